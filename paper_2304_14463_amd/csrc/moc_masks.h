// Predicates as lane masks, shared by the kernels of the evaluation, the staged evaluation, decode, toggles and the best
// single-field move.
#pragma once

#include "moc_cover.h"

namespace {

// ------------------------------------------------------------------ LDS by byte address
// The dynamic LDS segment starts at address 0 (the kernels declare no static LDS, which the
// host verifies before the first launch) and the node records are its first array: the LDS
// address of a record is its word index times 4 and needs no base register.
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
__device__ __forceinline__ uint32_t lds_read(uint32_t addr) { return *(const lds_u32*)(uintptr_t)addr; }
__device__ __forceinline__ uint2 lds_read2(uint32_t addr) {
  const u32x2 v = *(const lds_u32x2*)(uintptr_t)addr;
  return make_uint2(v.x, v.y);
}
typedef __attribute__((address_space(3))) uint16_t lds_u16;
__device__ __forceinline__ uint32_t lds_read_u16(uint32_t addr) { return *(const lds_u16*)(uintptr_t)addr; }

// Lane masks.  A predicate over the wave is one 64-bit scalar: a vector compare writes it
// directly, the scalar unit combines and counts them, and nothing per lane is spent on
// booleans.  The compares that pick a 16-bit half or a byte of their operand are written out
// (sub-dword operand selects) since the compiler would first extract the field into a register.
// Lanes that are switched off read as 0.  Use in wave-uniform control flow only.
#define MOC_MASK_CMP(name, text, breg)                                             \
  __device__ __forceinline__ lanemask name(uint32_t a, uint32_t b) {               \
    lanemask m;                                                                    \
    asm(text : "=s"(m) : "v"(a), breg(b));                                         \
    return m;                                                                      \
  }
MOC_MASK_CMP(u_lt, "v_cmp_lt_u32_e64 %0, %1, %2", "v")
MOC_MASK_CMP(u_le, "v_cmp_le_u32_e64 %0, %1, %2", "v")
MOC_MASK_CMP(u_eq, "v_cmp_eq_u32_e64 %0, %1, %2", "v")
MOC_MASK_CMP(i_gt, "v_cmp_gt_i32_e64 %0, %1, %2", "v")
// b the same in every lane (a scalar register)
MOC_MASK_CMP(u_lt_k, "v_cmp_lt_u32_e64 %0, %1, %2", "s")
#undef MOC_MASK_CMP
#define MOC_BYTE_CMP(name, sel)                                                                   \
  template <typename F>                                                                           \
  __device__ __forceinline__ lanemask name(F a, uint32_t b) {                                     \
    lanemask m;                                                                                   \
    asm("v_cmp_ne_u32_sdwa %0, %1, %2 src0_sel:" sel " src1_sel:DWORD" : "=s"(m) : "v"(a), "s"(b)); \
    return m;                                                                                     \
  }
MOC_BYTE_CMP(byte0_ne_k, "BYTE_0")
MOC_BYTE_CMP(byte1_ne_k, "BYTE_1")
MOC_BYTE_CMP(byte2_ne_k, "BYTE_2")
MOC_BYTE_CMP(byte3_ne_k, "BYTE_3")
MOC_BYTE_CMP(low_ne_k, "WORD_0")
MOC_BYTE_CMP(high_ne_k, "WORD_1")
#undef MOC_BYTE_CMP
// of a copy packed as s | e << 16: s < x and e >= y
__device__ __forceinline__ lanemask spans_lanes(uint32_t packed, uint32_t x, uint32_t y) {
  lanemask below, reaches;
  asm("v_cmp_lt_u32_sdwa %0, %1, %2 src0_sel:WORD_0 src1_sel:DWORD" : "=s"(below) : "v"(packed), "v"(x));
  asm("v_cmp_ge_u32_sdwa %0, %1, %2 src0_sel:WORD_1 src1_sel:DWORD" : "=s"(reaches) : "v"(packed), "v"(y));
  return below & reaches;
}
// it covers position x
__device__ __forceinline__ lanemask covers_lanes(uint32_t packed, uint32_t x) { return spans_lanes(packed, x, x); }
template <typename F>
__device__ __forceinline__ lanemask byte_ne_k(F a, int i, uint32_t b) {
  return i == 0 ? byte0_ne_k(a, b) : i == 1 ? byte1_ne_k(a, b) : i == 2 ? byte2_ne_k(a, b) : byte3_ne_k(a, b);
}
// per lane: m ? yes : no
__device__ __forceinline__ uint32_t pick(lanemask m, uint32_t yes, uint32_t no) {
  uint32_t r;
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(no), "v"(yes), "s"(m));
  return r;
}
// per lane: m ? yes : 0
__device__ __forceinline__ uint32_t pick(lanemask m, uint32_t yes) {
  uint32_t r;
  asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(yes), "s"(m));
  return r;
}
// per lane: x + 1 in the lanes of m, x in the others
__device__ __forceinline__ uint32_t add_lanes(lanemask m, uint32_t x) {
  uint32_t r;
  asm("v_addc_co_u32 %0, vcc, 0, %1, %2" : "=v"(r) : "v"(x), "s"(m) : "vcc");
  return r;
}
__device__ __forceinline__ int count(lanemask m) { return __builtin_popcountll(m); }
// true in exactly the lanes of m: `if (lanes(m))` runs its body with those lanes switched on
__device__ __forceinline__ bool lanes(lanemask m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// number of lanes of m below the calling lane, plus base
__device__ __forceinline__ uint32_t rank_in(lanemask m, uint32_t base) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}
// LDS[addr] = val in the lanes of m, without a branch: a branch would end the basic block, and
// 16-bit values that live across blocks are widened again where they are used.  LDS
// operations of a wave complete in order, so later reads see the write; the wave's count of
// outstanding LDS operations is only ever higher than the compiler assumes, never lower.
__device__ __forceinline__ void lds_write_lanes(lanemask m, uint32_t addr, uint32_t val) {
  lanemask saved;
  asm volatile("s_and_saveexec_b64 %0, %1\n\tds_write_b32 %2, %3\n\ts_mov_b64 exec, %0"
               : "=&s"(saved) : "s"(m), "v"(addr), "v"(val) : "memory", "scc");
}
// The low (HALF = 0) or high half of val, 16 bits wide; wait_for_lds_writes() before the barrier behind it.
template <int HALF>
__device__ __forceinline__ void lds_write16_lanes(lanemask m, uint32_t addr, uint32_t val) {
  lanemask saved;
  if constexpr (HALF == 0)
    asm volatile("s_and_saveexec_b64 %0, %1\n\tds_write_b16 %2, %3\n\ts_mov_b64 exec, %0"
                 : "=&s"(saved) : "s"(m), "v"(addr), "v"(val) : "memory", "scc");
  else
    asm volatile("s_and_saveexec_b64 %0, %1\n\tds_write_b16_d16_hi %2, %3\n\ts_mov_b64 exec, %0"
                 : "=&s"(saved) : "s"(m), "v"(addr), "v"(val) : "memory", "scc");
}
// The compiler does not count the writes above: it may see nothing to wait for at a barrier.
__device__ __forceinline__ void wait_for_lds_writes() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace
