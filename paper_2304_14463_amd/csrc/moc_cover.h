// The test of Eq. (5) on lane masks, shared by the evaluation kernels.
#pragma once

#include "moc_internal.h"

namespace {

using lanemask = uint64_t;   // a predicate over the 64 lanes of a wave

// The copies of a node as packed words s | e << 16 (MOC_DEAD if not live).
template <int CT>
struct Record {
  uint32_t w[CT];
};

// Eq. (5) for one copy of the consumer, packed as s | e << 16 in pv, against the CT copies of
// the provider in pu: adds to viol the number of lanes in which the copy is live and no copy of
// the provider has s_u + 1 <= s_v <= e_u (a dead copy has s = 0xFFFF and covers nothing).
// One block of instructions that ends in the count, so that three masks exist at a time
// however the surrounding code is scheduled: the masks of many edges in flight at once do not
// fit the scalar registers.
#define MOC_COVER_FIRST(U)                                                        \
  "v_cmp_lt_u32_sdwa %1, " U ", %5 src0_sel:WORD_0 src1_sel:WORD_0\n\t"           \
  "v_cmp_ge_u32_sdwa %2, " U ", %5 src0_sel:WORD_1 src1_sel:WORD_0\n\t"           \
  "s_and_b64 %1, %1, %2\n\t"
#define MOC_COVER_NEXT(U)                                                         \
  "v_cmp_lt_u32_sdwa %2, " U ", %5 src0_sel:WORD_0 src1_sel:WORD_0\n\t"           \
  "v_cmp_ge_u32_sdwa %3, " U ", %5 src0_sel:WORD_1 src1_sel:WORD_0\n\t"           \
  "s_and_b64 %2, %2, %3\n\t"                                                      \
  "s_or_b64 %1, %1, %2\n\t"
#define MOC_COVER_LAST                                                            \
  "v_cmp_ne_u32_sdwa %2, %5, %6 src0_sel:WORD_0 src1_sel:DWORD\n\t"               \
  "s_andn2_b64 %1, %2, %1\n\t"                                                    \
  "v_addc_co_u32 %0, vcc, 0, %0, %1"
// the same with "live" read off the word itself: a staged copy is live iff s <= e
#define MOC_COVER_LAST_SE                                                         \
  "v_cmp_le_u32_sdwa %2, %5, %5 src0_sel:WORD_0 src1_sel:WORD_1\n\t"              \
  "s_andn2_b64 %1, %2, %1\n\t"                                                    \
  "v_addc_co_u32 %0, vcc, 0, %0, %1"
#define MOC_COVER_REGS "+v"(viol), "=&s"(t1), "=&s"(t2), "=&s"(t3), "=&s"(c) : "v"(pv), "s"(dead)
template <int CT>
__device__ __forceinline__ void count_live_uncovered(int& viol, const Record<CT>& pu, uint32_t pv) {
  lanemask t1, t2, t3;
  int c;
  const uint32_t dead = MOC_DEAD;
  if constexpr (CT == 1)
    asm(MOC_COVER_FIRST("%7") MOC_COVER_LAST : MOC_COVER_REGS, "v"(pu.w[0]) : "scc", "vcc");
  else if constexpr (CT == 2)
    asm(MOC_COVER_FIRST("%7") MOC_COVER_NEXT("%8") MOC_COVER_LAST : MOC_COVER_REGS, "v"(pu.w[0]), "v"(pu.w[1]) : "scc", "vcc");
  else if constexpr (CT == 3)
    asm(MOC_COVER_FIRST("%7") MOC_COVER_NEXT("%8") MOC_COVER_NEXT("%9") MOC_COVER_LAST_SE
        : MOC_COVER_REGS, "v"(pu.w[0]), "v"(pu.w[1]), "v"(pu.w[2]) : "scc", "vcc");
  else if constexpr (CT == 5)
    asm(MOC_COVER_FIRST("%7") MOC_COVER_NEXT("%8") MOC_COVER_NEXT("%9") MOC_COVER_NEXT("%10") MOC_COVER_NEXT("%11") MOC_COVER_LAST_SE
        : MOC_COVER_REGS, "v"(pu.w[0]), "v"(pu.w[1]), "v"(pu.w[2]), "v"(pu.w[3]), "v"(pu.w[4]) : "scc", "vcc");
  else
    asm(MOC_COVER_FIRST("%7") MOC_COVER_NEXT("%8") MOC_COVER_NEXT("%9") MOC_COVER_NEXT("%10") MOC_COVER_LAST_SE
        : MOC_COVER_REGS, "v"(pu.w[0]), "v"(pu.w[1]), "v"(pu.w[2]), "v"(pu.w[3]) : "scc", "vcc");
}
// The same as a lane mask.
#define MOC_COVER_MASK                                                            \
  "v_cmp_le_u32_sdwa %1, %3, %3 src0_sel:WORD_0 src1_sel:WORD_1\n\t"              \
  "s_andn2_b64 %0, %1, %0"
#define MOC_COVER_M1(U)                                                           \
  "v_cmp_lt_u32_sdwa %0, " U ", %3 src0_sel:WORD_0 src1_sel:WORD_0\n\t"           \
  "v_cmp_ge_u32_sdwa %1, " U ", %3 src0_sel:WORD_1 src1_sel:WORD_0\n\t"           \
  "s_and_b64 %0, %0, %1\n\t"
#define MOC_COVER_M(U)                                                            \
  "v_cmp_lt_u32_sdwa %1, " U ", %3 src0_sel:WORD_0 src1_sel:WORD_0\n\t"           \
  "v_cmp_ge_u32_sdwa %2, " U ", %3 src0_sel:WORD_1 src1_sel:WORD_0\n\t"           \
  "s_and_b64 %1, %1, %2\n\t"                                                      \
  "s_or_b64 %0, %0, %1\n\t"
template <int CT>
__device__ __forceinline__ lanemask live_uncovered_lanes(const Record<CT>& pu, uint32_t pv) {
  lanemask m, t1, t2;
  if constexpr (CT == 1)
    asm(MOC_COVER_M1("%4") MOC_COVER_MASK : "=&s"(m), "=&s"(t1), "=&s"(t2) : "v"(pv), "v"(pu.w[0]) : "scc");
  else if constexpr (CT == 2)
    asm(MOC_COVER_M1("%4") MOC_COVER_M("%5") MOC_COVER_MASK : "=&s"(m), "=&s"(t1), "=&s"(t2) : "v"(pv), "v"(pu.w[0]), "v"(pu.w[1]) : "scc");
  else if constexpr (CT == 3)
    asm(MOC_COVER_M1("%4") MOC_COVER_M("%5") MOC_COVER_M("%6") MOC_COVER_MASK
        : "=&s"(m), "=&s"(t1), "=&s"(t2) : "v"(pv), "v"(pu.w[0]), "v"(pu.w[1]), "v"(pu.w[2]) : "scc");
  else
    asm(MOC_COVER_M1("%4") MOC_COVER_M("%5") MOC_COVER_M("%6") MOC_COVER_M("%7") MOC_COVER_MASK
        : "=&s"(m), "=&s"(t1), "=&s"(t2) : "v"(pv), "v"(pu.w[0]), "v"(pu.w[1]), "v"(pu.w[2]), "v"(pu.w[3]) : "scc");
  return m;
}
#undef MOC_COVER_MASK
#undef MOC_COVER_M1
#undef MOC_COVER_M
#undef MOC_COVER_FIRST
#undef MOC_COVER_NEXT
#undef MOC_COVER_LAST
#undef MOC_COVER_LAST_SE
#undef MOC_COVER_REGS

}  // namespace
