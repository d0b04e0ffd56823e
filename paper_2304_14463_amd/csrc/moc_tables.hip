// moc_eval_toggles, moc_eval_cuts, moc_eval_cuts_keep: every move of one kind of every base, one
// workgroup per base at a time (gfx950).  The base is staged in LDS (moc_moves.h) and every move is
// scored from it with the result moc_eval_batch has for the edited candidate.
#include <algorithm>

#include "moc_cut_moves.h"
#include "moc_masks.h"

namespace {

// ------------------------------------------------------------------ toggles
// A flip of one active flag.  A copy that is not well formed only starts or stops counting as such;
// a well-formed one joins or leaves the live copies of its node: the order pairs of the node change
// (Eq. (3)), its start is one more or one less (Eq. (6)), its inputs count or do not, consumers
// that only it covers lose their input, uncovered ones gain it (Eq. (5)), and the profile rises or
// falls on its interval (Eq. (4)).
//
// What Eq. (5) contributes is collected by a pass over the edges, one lane per edge (u, v), instead
// of a walk over both edge lists of every copy's node: for each copy of v, live or to be, one look
// at the copies of u says whether it has its input, and if a live copy of v has it from exactly one
// copy of u, or from none, what the flips of u's copies do to it.  The pass is the same length in
// every lane, needs no adjacency lists in LDS, and counts the base's own violations of Eq. (5) on
// its way.
//
// A staged copy that is well formed and not active carries bit 15 on top of its start (positions
// stay below 2^15: LDS bounds T), which keeps it from covering anything.
//
// Bound by the vector ALU (69 %) and LDS latency.  n = 2000, C = 2, 2048 bases: 475 us with a walk per copy
// over adjacency lists kept in LDS (one workgroup per compute unit), 112 us with the edges' conditions in
// vector registers and the positions at the ends of an interval picked by compares, 102 us now (calls on the
// same bases one behind the other; 109 on bases that are new to the caches).
constexpr uint32_t kOff = 0x8000u;

template <int CT, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT >= 512 ? 8 : 4))) void toggles_kernel(GraphView g, int64_t B, const int32_t* __restrict__ starts,
                                                     const int32_t* __restrict__ ends,
                                                     const uint8_t* __restrict__ active,
                                                     moc_toggle_score* __restrict__ out, MvLayout lay) {
  extern __shared__ uint32_t lds_raw[];
  constexpr int NW = NT / kWave, kAhead = 4;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int T = g.T, C = CT ? CT : g.C;
  BaseLds L;
  L.carve(lds_raw, lay);
  int32_t* const delta = reinterpret_cast<int32_t*>(L.extra);   // per copy: what a flip does to Eq. (5)

  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const int64_t row = b * T;
    // ---- stage: as stage_copies (moc_moves.h), the inactive copies kept as well
    const char* const s_row = reinterpret_cast<const char*>(starts + row);
    const char* const e_row = reinterpret_cast<const char*>(ends + row);
    const uint8_t* const a_row = active + row;
    int as[kAhead], ae[kAhead];
    uint32_t aa[kAhead];
    int2 asd[kAhead];
    {
      int own = t;   // offsets formed here for every base, not kept in registers across the bases
      asm volatile("" : "+v"(own));
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        const uint32_t k = (uint32_t)min(j * NT + own, T - 1);
        as[j] = *reinterpret_cast<const int32_t*>(s_row + 4u * k);
        ae[j] = *reinterpret_cast<const int32_t*>(e_row + 4u * k);
        aa[j] = a_row[k];
        asd[j] = g.size_dur[k / (uint32_t)C];
      }
    }
    for (int x = 4 * t; x < lay.blocks * kBlk; x += 4 * NT) *reinterpret_cast<int4*>(L.profile + x) = make_int4(0, 0, 0, 0);
    for (int x = t; x < T; x += NT) delta[x] = 0;
    for (int w = t; w < lay.bit_words; w += NT) { L.occ1[w] = 0; L.occ2[w] = 0; }
    __syncthreads();
    int viol = 0, live = 0, dur = 0;
    auto stage = [&](int k, int s, int e, uint32_t flag, int2 sd) {
      const bool act = flag != 0, well = (uint32_t)s <= (uint32_t)e && (uint32_t)e < (uint32_t)T;
      L.packed[k] = well ? (uint32_t)s | (uint32_t)e << 16 | (act ? 0u : kOff) : act ? MOC_DEAD | 0x10000u : MOC_DEAD;
      if (k % C == 0 && !act) ++viol;   // Eq. (7)
      if (act) dur += sd.y;
      if (act && !well) ++viol;         // Eq. (2)/(8)
      if (act && well) {
        ++live;
        atomicAdd(&L.profile[s], sd.x);
        if (e + 1 < T) atomicSub(&L.profile[e + 1], sd.x);
        const uint32_t bit = 1u << (s & 31);
        const uint32_t old = atomicOr(&L.occ1[s >> 5], bit);
        if (old & bit) atomicOr(&L.occ2[s >> 5], bit);
      }
    };
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int k = j * NT + t;
      if (k < T) stage(k, as[j], ae[j], aa[j], asd[j]);
    }
    for (int k = kAhead * NT + t; k < T; k += NT)
      stage(k, starts[row + k], ends[row + k], a_row[k], g.size_dur[k / C]);
    __syncthreads();
    // ---- Eq. (5), one lane per edge; which copies cover what as lane masks, `in` the lanes that have an edge
    // (One copy: there is nothing to combine, and conditions in vector registers are quicker: n = 60, 1024 bases 9.5
    // us, 10.2 with lane masks; n = 300, 512 bases 11.4 and 11.9.)
    auto edge = [&](uint32_t pair, lanemask in) {
      if constexpr (CT == 1) {
        const uint32_t pu = L.packed[pair & 0xFFFFu], pv = L.packed[pair >> 16], low = pv & 0xFFFFu, s = low & ~kOff;
        if (!lanes(in) || low == 0xFFFFu) return;
        if (!covers1(pu, s)) {
          atomicAdd(&delta[pair >> 16], low & kOff ? 1 : -1);
          if (!(low & kOff)) {
            ++viol;
            if ((pu & 0xFFFFu) != 0xFFFFu && covers1(pu & ~kOff, s)) atomicSub(&delta[pair & 0xFFFFu], 1);
          }
        } else if (!(low & kOff)) {
          atomicAdd(&delta[pair & 0xFFFFu], 1);
        }
        return;
      }
      const uint32_t* const pu = L.packed + (pair & 0xFFFFu);
      const uint32_t* const pv = L.packed + (pair >> 16);
      for (int i = 0; i < C; ++i) {
        const uint32_t copy = pv[i], s = copy & (0xFFFFu & ~kOff);
        lanemask some = 0, several = 0;
        uint32_t who = 0;
        for (int j = 0; j < C; ++j) {
          const lanemask c = covers_lanes(pu[j], s);
          several |= some & c;
          some |= c;
          if (j > 0) who = pick(c, (uint32_t)j, who);
        }
        const lanemask well = low_ne_k(copy, 0xFFFFu) & in, off = __ballot((copy & kOff) != 0);
        // a live copy that has its input from one copy of u alone loses it with that one's flip
        if (lanes(well & some & ~several & ~off)) atomicAdd(&delta[(pair & 0xFFFFu) + who], 1);
        if (lanes(well & ~some)) {   // the copy has no input: its flip adds or takes away a violation
          const bool live = !(copy & kOff);
          atomicAdd(&delta[(pair >> 16) + i], live ? -1 : 1);
          if (live) {
            ++viol;
            for (int j = 0; j < C; ++j)   // and the copies of u that would serve it take it away
              if ((pu[j] & 0xFFFFu) != 0xFFFFu && covers1(pu[j] & ~kOff, s)) atomicSub(&delta[(pair & 0xFFFFu) + j], 1);
          }
        }
      }
    };
    for (int x0 = 0; x0 < g.m; x0 += 4 * NT) {
      uint32_t pair[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) pair[d] = g.edge_pair_c[min(x0 + d * NT + t, g.m - 1)];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int left = g.m - (x0 + d * NT + wave * kWave);   // the same in all lanes
        if (left <= 0) break;
        edge(pair[d], left >= kWave ? ~(lanemask)0 : ((lanemask)1 << left) - 1);
      }
    }
    // ---- the base's violations and duration; its profile
    for (int v = t; v < g.n; v += NT) {   // Eq. (3): each live copy against the next live copy of its node
      int end = -1;
      for (int i = 0; i < C; ++i) {
        const uint32_t p = L.packed[v * C + i];
        if (p & kOff) continue;
        viol += end > (int)(p & 0xFFFFu) ? 1 : 0;
        end = (int)(p >> 16);
      }
    }
    for (int w = t; w < lay.bit_words; w += NT) viol -= __popc(L.occ1[w]);   // Eq. (6): live copies - distinct starts
    viol = scan_sum(viol + live);
    dur = scan_sum(dur);
    if (lane == kWave - 1) {
      L.scratch[32 + wave] = viol;
      L.scratch[64 + wave] = dur;
    }
    scan_profile<NT>(L, lay, T, t);
    build_maxima<NT>(L, lay, t);
    int base_viol = 0, base_dur = 0;
    for (int w = 0; w < NW; ++w) {
      base_viol += L.scratch[32 + w];
      base_dur += L.scratch[64 + w];
    }
    base_viol = __builtin_amdgcn_readfirstlane(base_viol);
    base_dur = __builtin_amdgcn_readfirstlane(base_dur);
    const int base_peak = __builtin_amdgcn_readfirstlane(L.pre[lay.blocks]);
    // ---- one lane per copy
    for (int k = t; k < T; k += NT) {
      const int v = k / C, i = k - v * C;
      const uint32_t mine = L.packed[k];
      const bool well = (mine & 0xFFFFu) != 0xFFFFu, was = well ? !(mine & kOff) : mine != MOC_DEAD;
      const int s = (int)(mine & 0x7FFFu), e = (int)(mine >> 16);
      const int2 sd = g.size_dur[v];
      int vv = base_viol + (i != 0 ? 0 : was ? 1 : -1);   // Eq. (7)
      int pk = base_peak;
      if (!well) {
        vv += was ? -1 : 1;   // Eq. (2)/(8)
      } else {
        // Eq. (3) among the live copies of v, with and without copy k
        int with = 0, without = 0;
        if constexpr (CT == 2) {
          const uint32_t p = L.packed[k ^ 1];
          if (!(p & kOff)) with = i == 0 ? (e > (int)(p & 0xFFFFu) ? 1 : 0) : ((int)(p >> 16) > s ? 1 : 0);
        } else if constexpr (CT != 1) {
          int end_with = -1, end_without = -1;
          for (int j = 0; j < C; ++j) {
            const uint32_t p = L.packed[v * C + j];
            if ((p & kOff) && j != i) continue;   // not live (MOC_DEAD carries the bit as well)
            const int start = j == i ? s : (int)(p & 0xFFFFu), end = (int)(p >> 16);
            with += end_with > start ? 1 : 0;
            end_with = end;
            if (j != i) {
              without += end_without > start ? 1 : 0;
              end_without = end;
            }
          }
        }
        vv += (was ? without - with : with - without) + delta[k];
        // Eq. (6): a shared start loses one of its copies, or a taken start gains one
        if (was) vv -= bit_at(L.occ2, s) ? 1 : 0;
        else vv += bit_at(L.occ1, s) ? 1 : 0;
        const InOut m = range_maxima<true>(L, lay.blocks, s, e);
        pk = max(max(m.in + (was ? -sd.x : sd.x), 0), m.out);
      }
      moc_toggle_score sc;
      sc.violations = vv;
      sc.peak = pk;
      sc.duration = (int64_t)base_dur + (was ? -sd.y : sd.y);
      out[row + k] = sc;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ cuts
// The table, the best move, or both.  MODE 1: the cuts that keep the producer's inputs.  Bound by
// instruction issue and LDS latency: scoring a move is some hundred instructions in a chain of reads.
// n = 1000, C = 2, 2048 bases, plain cuts, table and best move: 303 us with one workgroup of 16 waves
// per compute unit (adjacency lists of 32-bit words, prefix and suffix maxima per position), 88 to
// 90 us now (on the same bases again and again; 94 to 96 on new ones); 126 us with the mode read at run time, whose
// registers cost a workgroup per compute unit.
template <int CT, int NT, bool LISTS, int MODE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 1024 ? 4 : 6))) void cuts_kernel(GraphView g, int64_t B, const int32_t* __restrict__ starts,
                                                  const int32_t* __restrict__ ends, const uint8_t* __restrict__ active,
                                                  moc_cut_score* __restrict__ out, moc_best_move* __restrict__ out_best,
                                                  MvLayout lay) {
  extern __shared__ uint32_t lds_raw[];
  constexpr int NW = NT / kWave;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int T = g.T, C = CT ? CT : g.C;
  BaseLds L;
  L.carve(lds_raw, lay);
  Lists<LISTS> lists;
  lists.template load<NT>(g, lds_raw + lay.lists, t);
  int32_t* const queue = reinterpret_cast<int32_t*>(L.extra);

  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const int64_t row = b * T;
    int own = t;   // what derives from the thread index is formed again for every base
    asm volatile("" : "+v"(own));
    const StageSums sums = stage_copies<CT, NT>(g, L, lay, starts + row, ends + row, active + row, own);
    int viol = sums.viol + sums.live + count_order_and_inputs<CT, NT>(g, lists, L.packed, own);
    for (int w = own; w < lay.bit_words; w += NT) viol -= __popc(L.occ1[w]);   // Eq. (6): live copies - distinct starts
    viol = scan_sum(viol);
    const int dur = scan_sum(sums.dur);
    if (lane == kWave - 1) {
      L.scratch[96 + wave] = viol;
      L.scratch[112 + wave] = dur;
    }
    clear_marks(L, own);
    scan_profile<NT>(L, lay, T, own);
    build_maxima<NT>(L, lay, own);
    int base_viol = 0, base_dur = 0;
    for (int w = 0; w < NW; ++w) {
      base_viol += L.scratch[96 + w];
      base_dur += L.scratch[112 + w];
    }
    base_viol = __builtin_amdgcn_readfirstlane(base_viol);
    base_dur = __builtin_amdgcn_readfirstlane(base_dur);
    const int base_peak = __builtin_amdgcn_readfirstlane(L.pre[lay.blocks]);
    const PeakCount at_peak = mark_peak<NT>(L, lay, T, base_peak, own);

    moc_cut_score* const table = out ? out + b * ((int64_t)g.m * C) : nullptr;
    BestCut best;
    score_cuts<CT, NT>(g, lists, L, lay, queue, MODE, base_viol, base_peak, at_peak, false, best, own,
                       [&](int q, int ub, const CutScore* sc) {
                         if (!table) return;
                         moc_cut_score r{-1, -1, 0};
                         if (sc) {
                           r.violations = sc->viol;
                           r.peak = sc->peak;
                           r.duration = (int64_t)base_dur + g.size_dur[ub / C].y;
                         }
                         table[q] = r;
                       });
    if (out_best) {
      best_of_workgroup<NT>(best, L.scratch, own);
      if (own == 0) {
        const bool none = best.move() < 0;
        out_best[b] = moc_best_move{best.move(), none ? 0 : best.viol(), none ? 0 : (int64_t)best.peak()};
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ host side
using TogglesKernel = void (*)(GraphView, int64_t, const int32_t*, const int32_t*, const uint8_t*, moc_toggle_score*, MvLayout);
using CutsKernel = void (*)(GraphView, int64_t, const int32_t*, const int32_t*, const uint8_t*, moc_cut_score*, moc_best_move*,
                            MvLayout);

template <int NT>
TogglesKernel pick_toggles(int C) {
  switch (C) {
    case 1: return toggles_kernel<1, NT>;
    case 2: return toggles_kernel<2, NT>;
    case 3: return toggles_kernel<3, NT>;
    case 4: return toggles_kernel<4, NT>;
    default: return toggles_kernel<0, NT>;
  }
}
template <int NT, bool LISTS, int MODE>
CutsKernel pick_cuts(int C) {
  switch (C) {
    case 2: return cuts_kernel<2, NT, LISTS, MODE>;
    case 3: return cuts_kernel<3, NT, LISTS, MODE>;
    default: return cuts_kernel<0, NT, LISTS, MODE>;
  }
}
template <int MODE>
CutsKernel pick_cuts(int C, int nt, bool lists) {
  if (!lists) return pick_cuts<1024, false, MODE>(C);
  return nt == 256 ? pick_cuts<256, true, MODE>(C) : nt == 512 ? pick_cuts<512, true, MODE>(C) : pick_cuts<1024, true, MODE>(C);
}

// Workgroups that share a compute unit: what LDS holds, or what the batch has for each unit.
int bases_together(const moc_graph* g, int64_t B, int bytes) {
  return (int)std::min<int64_t>(g->max_lds / bytes, (B + g->num_cu - 1) / g->num_cu);
}

template <typename K>
int resident_grid(const moc_graph* g, K kern, int nt, int bytes, int64_t B, unsigned* grid) {
  int per_cu = 0;
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), nt, bytes, false, &per_cu)) return rc;
  *grid = (unsigned)std::min<int64_t>(B, (int64_t)per_cu * g->num_cu);
  return MOC_OK;
}

int check_bases(const int32_t* starts, const int32_t* ends, const uint8_t* active) {
  if (!starts || !ends || !active) return MOC_EINVAL;
  if (((uintptr_t)starts | (uintptr_t)ends) & 3) return MOC_EINVAL;
  return MOC_OK;
}

int check_graph(const moc_graph* g) {
  int dev = -1;
  MOC_HIP(hipGetDevice(&dev));
  if (dev != g->device) return MOC_EDEVICE;
  if (g->has_self_loop) return MOC_EINVAL;
  if (!moves_fit(g->view.T, g->max_lds)) return MOC_EOVERFLOW;
  return MOC_OK;
}

int eval_cuts(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends, const uint8_t* active,
              int mode, moc_cut_score* out_moves, moc_best_move* out_best, void* hip_stream) {
  if (!g || B < 0) return MOC_EINVAL;
  if (!out_moves && !out_best) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (const int rc = check_bases(starts, ends, active)) return rc;
  if (((uintptr_t)out_moves & 7) || ((uintptr_t)out_best & 7)) return MOC_EINVAL;
  if (const int rc = moc_check_cuts(g)) return rc;
  const GraphView& v = g->view;
  const auto layout = [&](int nt) { return mv_layout(v.T, v.n, v.m, 2 * nt, true, g->max_lds); };
  // As many threads as fill the compute unit with the workgroups its LDS holds and the batch has for it
  // (87 keeping bases of n = 558, one per unit: 613 us before, about 630 by the LDS rule alone, 343 now).
  // Plain cuts, C = 2, by
  // 256 / 512 / 1024 threads: n = 442 (six fit), 2048 bases 68 / 74 / 132 us; n = 1000 (three),
  // 2048 bases 116 / 90 / 149 us; n = 2000 (one), 1024 bases 463 / 269 / 200 us.  Without the lists
  // in LDS one workgroup fits anyway.
  const int together = bases_together(g, B, layout(256).bytes);
  const int nt = !layout(1024).lists || together <= 1 ? 1024 : together <= 3 ? 512 : 256;
  const MvLayout lay = layout(nt);
  if (lay.bytes > g->max_lds) return MOC_EOVERFLOW;
  const CutsKernel kern = mode == 0 ? pick_cuts<0>(v.C, nt, lay.lists != 0) : pick_cuts<1>(v.C, nt, lay.lists != 0);
  unsigned grid = 0;
  if (const int rc = resident_grid(g, kern, nt, lay.bytes, B, &grid)) return rc;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lay.bytes, static_cast<hipStream_t>(hip_stream), v, B, starts, ends, active,
                     out_moves, out_best, lay);
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

}  // namespace

int moc_check_cuts(const moc_graph* g) {
  if (const int rc = check_graph(g)) return rc;
  if ((int64_t)g->view.m * g->view.C > 0x7FFFFFFFll) return MOC_EOVERFLOW;
  return MOC_OK;
}

extern "C" int moc_eval_toggles(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends,
                                const uint8_t* active, moc_toggle_score* out, void* hip_stream) {
  if (!g || B < 0) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (!out || ((uintptr_t)out & 7)) return MOC_EINVAL;
  if (const int rc = check_bases(starts, ends, active)) return rc;
  if (const int rc = check_graph(g)) return rc;
  const GraphView& v = g->view;
  const MvLayout lay = mv_layout(v.T, v.n, v.m, v.T, false, g->max_lds);
  if (lay.bytes > g->max_lds) return MOC_EOVERFLOW;
  // Threads as above; the kernel is held to 64 registers where that lets two workgroups of 1024 in.
  // n = 2000, C = 2 (two fit), 2048 bases: 165 us with 256 threads, 122 with 512, 112 with 1024 (102 on the
  // present kernel).
  const int together = bases_together(g, B, lay.bytes);
  const int nt = together <= 2 ? 1024 : together <= 4 ? 512 : 256;
  const TogglesKernel kern = nt == 1024 ? pick_toggles<1024>(v.C) : nt == 512 ? pick_toggles<512>(v.C) : pick_toggles<256>(v.C);
  unsigned grid = 0;
  if (const int rc = resident_grid(g, kern, nt, lay.bytes, B, &grid)) return rc;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lay.bytes, static_cast<hipStream_t>(hip_stream), v, B, starts, ends, active,
                     out, lay);
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

extern "C" int moc_eval_cuts(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends,
                             const uint8_t* active, moc_cut_score* out_moves, moc_best_move* out_best,
                             void* hip_stream) {
  return eval_cuts(g, B, starts, ends, active, 0, out_moves, out_best, hip_stream);
}

extern "C" int moc_eval_cuts_keep(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends,
                                  const uint8_t* active, moc_cut_score* out_moves, moc_best_move* out_best,
                                  void* hip_stream) {
  return eval_cuts(g, B, starts, ends, active, 1, out_moves, out_best, hip_stream);
}
