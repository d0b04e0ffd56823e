// The second phase of moc_search_two_phase: merges that lower the duration of a candidate within
// the budget, one workgroup per candidate from its first step to its last (gfx950).
//
// A merge switches a live copy c off and keeps b, the nearest live copy of its node below it,
// until the later of the two ends.  What changes is the node's own order (Eq. (3)), the start and
// the inputs of c (Eq. (5), (6)), which copies serve the node's consumers (Eq. (5)), and the
// profile on one stretch: +m between the two copies, or -m where they overlapped.  So the base is
// staged once -- packed copies, profile with range maxima (moc_moves.h) -- and a merge is scored
// by one lane from it, with the result moc_eval_batch has for the edited candidate.
#include "moc_moves.h"

namespace {

struct Merge { int c, below; };

// The nearest live copy of the node of copy k below k, -1 if none; `packed` as staged.
// (The same number of rounds in every lane: the answer goes into a ballot.)
__device__ __forceinline__ int live_below(const uint32_t* __restrict__ packed, int C, int k) {
  const int first = k - k % C;
  int found = -1;
  for (int i = 0; i + 1 < C; ++i)
    if (first + i < k && live_of(packed[first + i])) found = first + i;
  return found;
}

// The stretch of the profile the merge changes, and by how much per unit of m_v (0: nothing).
__device__ __forceinline__ Range merged_range(uint32_t pc, uint32_t pb, int size) {
  const int sc = (int)(pc & 0xFFFFu), ec = (int)(pc >> 16), eb = (int)(pb >> 16);
  if (sc > eb) return Range{eb + 1, sc - 1, sc - 1 > eb ? size : 0};
  return Range{sc, min(ec, eb), -size};
}

// One workgroup per candidate, a step per merge applied: list the copies that have a merge, in
// index order, as many as K; one lane per entry scores it; the feasible one of lowest duration,
// then peak, then index is applied to the staged base and to the candidate's rows.  What bounds a
// step is a chain of LDS latencies (list, walk over the node's edges, range maxima, tables), so
// the workgroup is small and several share a compute unit.  1024 walkers at n = 442, C = 2, up to
// 48 steps of K = 64: 0.25 ms.  (Every merge written out as a row of its own and evaluated by
// moc_eval_batch, four launches a step: 19 ms, of which 9.8 the writing and 7.9 the evaluation.)
template <int CT, int NT, bool LISTS>
__global__ __launch_bounds__(NT) void merge_kernel(GraphView g, int32_t* __restrict__ starts, int32_t* __restrict__ ends,
                                                   uint8_t* __restrict__ active, int K, int max_steps,
                                                   int32_t* __restrict__ merges, MvLayout lay) {
  extern __shared__ uint32_t lds_raw[];
  constexpr int NW = NT / kWave;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int T = g.T, C = CT ? CT : g.C;
  BaseLds L;
  L.carve(lds_raw, lay);
  Lists<LISTS> lists;
  lists.template load<NT>(g, lds_raw + lay.lists, t);
  uint64_t* const masks = reinterpret_cast<uint64_t*>(L.peak_bits);   // per 64 copies: those that have a merge
  uint16_t* const list = reinterpret_cast<uint16_t*>(L.extra);
  const int chunks = (T + kWave - 1) / kWave;
  const int64_t row = (int64_t)blockIdx.x * T;

  const StageSums sums = stage_copies<CT, NT>(g, L, lay, starts + row, ends + row, active + row, t);
  int viol = sums.viol + sums.live + count_order_and_inputs<CT, NT>(g, lists, L.packed, t);
  for (int w = t; w < lay.bit_words; w += NT) viol -= __popc(L.occ1[w]);   // Eq. (6): live copies - distinct starts
  viol = last_lane(scan_sum(viol));
  if (lane == 0) L.scratch[32 + wave] = viol;
  scan_profile<NT>(L, lay, T, t);
  build_maxima<NT>(L, lay, t);
  int base_viol = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) base_viol += L.scratch[32 + w];

  int steps = 0;
  for (; steps < max_steps; ++steps) {
    // ---- the list
    for (int c = wave; c < chunks; c += NW) {
      const int k = c * kWave + lane;
      const bool mergeable = k < T && live_of(L.packed[k]) && live_below(L.packed, C, k) >= 0;
      const uint64_t mask = __ballot(mergeable);
      if (lane == 0) masks[c] = mask;
    }
    __syncthreads();
    int count = 0;
    for (int c0 = 0; c0 < chunks; c0 += kWave) {   // every wave: the entries before each chunk, its own chunks written out
      const uint64_t mask = c0 + lane < chunks ? masks[c0 + lane] : 0;
      const int incl = count + scan_sum(__popcll(mask));
      for (int c = c0 + wave; c < min(c0 + kWave, chunks); c += NW) {
        const uint64_t m = masks[c];
        const int before = __builtin_amdgcn_readlane(incl, c - c0) - __popcll(m);
        if ((m >> lane) & 1) list[before + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)(c * kWave + lane);
      }
      count = last_lane(incl);
    }
    count = min(count, K);
    __syncthreads();

    // ---- one lane per entry.  key = (2^31 - 1 - w_v) << 32 | peak: the lowest duration, then the
    // lowest peak; then the lowest copy index.
    uint64_t best = ~0ull;
    int best_copy = 0x7FFFFFFF;
    for (int r = t; r < count; r += NT) {
      const int k = list[r];
      const int v = k / C, below = live_below(L.packed, C, k);
      const uint32_t pc = L.packed[k], pb = L.packed[below];
      const uint32_t sc = pc & 0xFFFFu;
      const uint32_t joined = (pb & 0xFFFFu) | (max(pb >> 16, pc >> 16) << 16);
      int vv = base_viol;
      // Eq. (3) among the live copies of v, before and after
      int end_before = -1, end_after = -1;
      for (int i = 0; i < C; ++i) {
        const uint32_t p = L.packed[v * C + i];
        if (!live_of(p)) continue;
        const int start = (int)(p & 0xFFFFu);
        vv -= end_before > start ? 1 : 0;
        end_before = (int)(p >> 16);
        if (v * C + i == k) continue;
        vv += end_after > start ? 1 : 0;
        end_after = (int)((v * C + i == below ? joined : p) >> 16);
      }
      if (bit_at(L.occ2, (int)sc)) --vv;   // Eq. (6): a shared start loses one of its copies
      // Eq. (5): the inputs of c are not asked for any more
      for (int x = lists.in_begin(v), x1 = lists.in_begin(v + 1); x < x1; ++x) {
        const uint32_t* const pu = L.packed + (lists.pair(x) & 0xFFFFu);
        bool held = false;
        for (int i = 0; i < C; ++i) held = held || covers1(pu[i], sc);
        vv -= held ? 0 : 1;
      }
      // Eq. (5): the consumers of v, served by the copies as they stand and as they would be
      for (int y = lists.out_begin(v), y1 = lists.out_begin(v + 1); y < y1; ++y) {
        const uint32_t* const pw = L.packed + lists.consumer_copy(y, C);
        for (int j = 0; j < C; ++j) {
          const uint32_t at = pw[j] & 0xFFFFu;
          if (at == 0xFFFFu) continue;
          bool others = false;
          for (int i = 0; i < C; ++i)
            others = others || (v * C + i != k && v * C + i != below && covers1(L.packed[v * C + i], at));
          if (others) continue;
          vv += (covers1(joined, at) ? 0 : 1) - (covers1(pc, at) || covers1(pb, at) ? 0 : 1);
        }
      }
      if (vv != 0) continue;
      const Range range = merged_range(pc, pb, lists.size_of(v));
      int peak = L.pre[lay.blocks];
      if (range.change != 0) {
        const InOut m = range_maxima<true>(L, lay.blocks, range.lo, range.hi);
        peak = max(m.in + range.change, m.out);
      }
      if ((int64_t)peak > g.budget) continue;
      const uint64_t key = (uint64_t)(0x7FFFFFFFu - (uint32_t)g.size_dur[v].y) << 32 | (uint32_t)peak;
      if (key < best || (key == best && k < best_copy)) {
        best = key;
        best_copy = k;
      }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)best, off);
      const int oc = __shfl_xor(best_copy, off);
      if (o < best || (o == best && oc < best_copy)) {
        best = o;
        best_copy = oc;
      }
    }
    if (lane == 0) {
      L.scratch[4 * wave] = (int)(uint32_t)best;
      L.scratch[4 * wave + 1] = (int)(uint32_t)(best >> 32);
      L.scratch[4 * wave + 2] = best_copy;
    }
    __syncthreads();
    best = ~0ull;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint64_t o = (uint64_t)(uint32_t)L.scratch[4 * w + 1] << 32 | (uint32_t)L.scratch[4 * w];
      const int oc = L.scratch[4 * w + 2];
      if (o < best || (o == best && oc < best_copy)) {
        best = o;
        best_copy = oc;
      }
    }
    if (best == ~0ull) break;   // no feasible merge: the candidate stays as it is
    // ---- apply it; the result has no violations
    const int k = __builtin_amdgcn_readfirstlane(best_copy);
    const int below = __builtin_amdgcn_readfirstlane(live_below(L.packed, C, k));
    const uint32_t pc = L.packed[k], pb = L.packed[below];
    const Range range = merged_range(pc, pb, g.size_dur[k / C].x);
    base_viol = 0;
    __syncthreads();
    if (t == 0) {
      const uint32_t end = max(pb >> 16, pc >> 16);
      L.packed[k] = MOC_DEAD;
      L.packed[below] = (pb & 0xFFFFu) | (end << 16);
      const uint32_t s = pc & 0xFFFFu;
      L.occ2[s >> 5] &= ~(1u << (s & 31));   // a shared start is shared no more (nothing is: no violations)
      ends[row + below] = (int32_t)end;
      active[row + k] = 0;
    }
    add_ranges<NT>(L, lay, &range, 1, t);
    if (range.change != 0) build_maxima<NT>(L, lay, t);
  }
  if (t == 0) merges[blockIdx.x] = steps;
}

using MergeKernel = void (*)(GraphView, int32_t*, int32_t*, uint8_t*, int, int, int32_t*, MvLayout);

template <int NT, bool LISTS>
MergeKernel pick_merge(int C) {
  switch (C) {
    case 2: return merge_kernel<2, NT, LISTS>;
    case 3: return merge_kernel<3, NT, LISTS>;
    case 4: return merge_kernel<4, NT, LISTS>;
    default: return merge_kernel<0, NT, LISTS>;
  }
}

}  // namespace

int moc_queue_merges(const moc_graph* g, int64_t B, int32_t* starts, int32_t* ends, uint8_t* active, int max_steps, int K,
                     int32_t* out_merges, hipStream_t stream) {
  const int T = g->view.T;
  const MvLayout lay = mv_layout(T, g->view.n, g->view.m, (T + 1) / 2, true, g->max_lds);
  if (lay.bytes > g->max_lds) return MOC_EOVERFLOW;
  constexpr int NT = 256;
  const MergeKernel kern = lay.lists ? pick_merge<NT, true>(g->view.C) : pick_merge<NT, false>(g->view.C);
  int per_cu = 0;   // not used: the call is for the kernel's LDS limit
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), NT, lay.bytes, false, &per_cu)) return rc;
  hipLaunchKernelGGL(kern, dim3((unsigned)B), dim3(NT), lay.bytes, stream, g->view, starts, ends, active, K, max_steps,
                     out_merges, lay);
  return MOC_OK;
}
