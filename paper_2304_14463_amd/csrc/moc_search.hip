// The searches that change a candidate by cuts (moc_search_cuts, the first phase of
// moc_search_two_phase) and by merges (its second phase), one workgroup per candidate from its
// first step to its last (gfx950).
//
// The base is staged once -- packed copies, profile with range maxima (moc_moves.h) -- and stays in
// LDS: a step scores the moves, eight lanes each, chooses, edits the candidate's rows and the staged
// base alike, and brings the maxima up to date.  Nothing is read from global memory between two
// steps, and a candidate that has come to its end costs nothing more.
//
// Cuts: see moc_cut_moves.h.  A merge switches a live copy c off and keeps b, the nearest live copy of its node below it,
// until the later of the two ends.  What changes is the node's own order (Eq. (3)), the start and
// the inputs of c (Eq. (5), (6)), which copies serve the node's consumers (Eq. (5)), and the
// profile on one stretch: +m between the two copies, or -m where they overlapped.
#include <algorithm>

#include "moc_cut_moves.h"

namespace {

static_assert(kMaxRanges == kWave + 1 && kCutWords == (int)(sizeof(Cut) / 4), "descend_words");

// One workgroup per candidate: up to max_steps cuts, each the best of the candidate as it stands,
// applied if it lowers (violations, max(peak, M)) or, above the budget with both unchanged, leaves
// fewer positions at the peak.  A step is a chain of short phases; 1024 walkers at n = 442 (four to a compute
// unit) are bound by the vector instructions of all of them together, 77 % busy, a few walkers by the chain:
// 13.6 us with cuts that keep inputs (sieve 6, scoring 3.5, edit 2, tables 1; 21 to 25 with one lane per
// move), 8 with plain cuts at n = 1000 (sieve 1.5, scoring 1.6, edit 1.3, tables 1.4; 13).  The walkers are
// all resident, so the launch lasts as long as those with the most steps: n = 442, 1024 walkers, up to 64
// keeping cuts 0.40 and 0.7 ms for two sets of inputs (0.76 and 1.36 with one lane per move; 27 ms with two
// launches a step that staged and scored everything again); n = 1000, 32 walkers, 32 plain cuts: 0.27 ms
// (0.42; 1.31).
template <int CT, int NT, bool LISTS, int MODE, bool WIDE>
__global__ __launch_bounds__(NT) void descend_cuts_kernel(GraphView g, int32_t* __restrict__ starts, int32_t* __restrict__ ends,
                                                          uint8_t* __restrict__ active, int max_steps,
                                                          moc_best_move* __restrict__ last_move, int32_t* __restrict__ out_steps,
                                                          int cap, MvLayout lay) {
  extern __shared__ uint32_t lds_raw[];
  constexpr int NW = NT / kWave;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int T = g.T, C = CT ? CT : g.C;
  BaseLds L;
  L.carve(lds_raw, lay);
  Lists<LISTS> lists;
  lists.template load<NT>(g, lds_raw + lay.lists, t);
  int32_t* const queue = reinterpret_cast<int32_t*>(L.extra);
  Range* const ranges = reinterpret_cast<Range*>(queue + 2 * kWave * NW);
  int32_t* const n_ranges = reinterpret_cast<int32_t*>(ranges + kMaxRanges);
  Cut* const chosen_cut = reinterpret_cast<Cut*>(n_ranges + 1);
  const SiftLds sift = carve_sift(L.extra + descend_words(NT), cap);
  const int64_t row = (int64_t)blockIdx.x * T;

  const StageSums sums = stage_copies<CT, NT>(g, L, lay, starts + row, ends + row, active + row, t);
  int viol = sums.viol + sums.live + count_order_and_inputs<CT, NT>(g, lists, L.packed, t);
  for (int w = t; w < lay.bit_words; w += NT) viol -= __popc(L.occ1[w]);   // Eq. (6): live copies - distinct starts
  viol = last_lane(scan_sum(viol));
  if (lane == 0) L.scratch[128 + wave] = viol;
  clear_marks(L, t);
  scan_profile<NT>(L, lay, T, t);
  build_maxima<NT>(L, lay, t);
  int base_viol = 0, base_peak = L.pre[lay.blocks];
#pragma unroll
  for (int w = 0; w < NW; ++w) base_viol += L.scratch[128 + w];

  int steps = 0;
  moc_best_move chosen{-1, 0, 0};
  clear_sift<NT>(sift, t);
  PeakCount at_peak = mark_peak<NT>(L, lay, T, base_peak, t);
  for (; steps < max_steps; ++steps) {
    chosen = moc_best_move{-1, 0, 0};
    if (base_viol == 0 && (int64_t)base_peak <= g.budget) break;   // no move lowers anything a step looks at
    BestCut best;
    Cut cut{};
    bool known = false;   // this lane holds the chosen move in `cut`
    if (base_viol != 0 || !best_cut_of_clean_base<CT, NT, MODE, WIDE>(g, lists, L, lay, sift, base_peak, at_peak, best, cut, known, t)) {
      best = BestCut{};
      known = false;
      score_cuts<CT, NT>(g, lists, L, lay, queue, MODE, base_viol, base_peak, at_peak, base_viol == 0, best, t,
                         [](int, int, const CutScore*) {});
      best_of_workgroup<NT>(best, L.scratch, t);
      if (t == 0 && best.move() >= 0) {
        const int x = best.move() / C;
        const uint32_t pair = lists.pair(x);
        known = find_cut(lists, C, L, (int)(pair & 0xFFFFu), (int)(L.packed[(pair >> 16) + best.move() - x * C] & 0xFFFFu), MODE,
                         base_viol == 0, cut);
      }
    }
    const int q = best.move();
    if (q < 0) break;
    const int64_t now = max((int64_t)base_peak, g.budget), then = max((int64_t)best.peak(), g.budget);
    if (!(best.viol() < base_viol ||
          (best.viol() == base_viol &&
           (then < now || (then == now && (int64_t)base_peak > g.budget && best.at() < at_peak.total)))))
      break;
    chosen = moc_best_move{q, best.viol(), (int64_t)best.peak()};

    // ---- apply it: one wave edits the copies and lists the stretches of the profile that change
    if (known) *chosen_cut = cut;
    begin_marks<NT>(L, lay, t);
    clear_sift<NT>(sift, t);
    __syncthreads();
    cut = *chosen_cut;
    const int ub = (int)(lists.pair(q / C) & 0xFFFFu), u = ub / C;
    const int y0 = lists.in_begin(u), y1 = lists.in_begin(u + 1);
    const int rounds = MODE == 1 ? max(1, (y1 - y0 + kWave - 1) / kWave) : 1;
    for (int round = 0; round < rounds; ++round) {
      __syncthreads();   // every wave has read what it needs of the copies, the stretches of the last round are added
      if (wave == 0) {
        int count = 0;
        if (round == 0) {
          if (lane == 0) ranges[0] = Range{cut.last_use + 1, cut.p - 1, -lists.size_of(u)};
          count = 1;
        }
        int kept = -1, end = -1, w = 0;   // the copy of the lane's predecessor of u that is kept until p
        if (MODE == 1) {
          const int y = y0 + round * kWave + lane;
          if (y < y1) {
            w = (int)(lists.pair(y) & 0xFFFFu);
            int held = 0;
            for (int c = 0; c < C; ++c) {
              const uint32_t pw = L.packed[w + c];
              held |= covers1(pw, (uint32_t)cut.p) ? 1 : 0;
              if (live_of(pw) && (int)(pw >> 16) < cut.p && (int)(pw >> 16) >= end) {
                kept = c;
                end = (int)(pw >> 16);
              }
            }
            if (held) kept = -1;
            // listed before among these 64 (among earlier ones: it is held by now)
            for (int z = y0 + round * kWave; z < y; ++z)
              if ((int)(lists.pair(z) & 0xFFFFu) == w) kept = -1;
          }
          const uint64_t m = __ballot(kept >= 0);
          wave_lds_order();   // all lanes have read the copies
          if (kept >= 0) {
            ranges[count + __popcll(m & ((1ull << lane) - 1))] = Range{end + 1, cut.p, lists.size_of(w / C)};
            L.packed[w + kept] = (L.packed[w + kept] & 0xFFFFu) | (uint32_t)cut.p << 16;
            ends[row + w + kept] = cut.p;
          }
          count += __popcll(m);
        }
        if (lane == 0) {
          *n_ranges = count;
          if (round == rounds - 1) {
            L.packed[ub + cut.k] = (uint32_t)cut.sk | (uint32_t)cut.last_use << 16;
            L.packed[ub + cut.j] = (uint32_t)cut.p | (uint32_t)cut.ek << 16;
            L.occ1[cut.p >> 5] |= 1u << (cut.p & 31);
            ends[row + ub + cut.k] = cut.last_use;
            starts[row + ub + cut.j] = cut.p;
            ends[row + ub + cut.j] = cut.ek;
            active[row + ub + cut.j] = 1;
          }
        }
      }
      __syncthreads();
      if (round == rounds - 1) add_ranges<NT, true>(L, lay, ranges, *n_ranges, best.peak(), T, t);
      else add_ranges<NT, false>(L, lay, ranges, *n_ranges, 0, T, t);
    }
    build_maxima<NT>(L, lay, t);
    base_viol = best.viol();
    base_peak = best.peak();
    at_peak = count_marks<NT>(L, lay, t);
  }
  if (t == 0) {
    out_steps[blockIdx.x] = steps;
    last_move[blockIdx.x] = chosen;
  }
}

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
// index order, as many as K; eight lanes per entry score it; the feasible one of lowest duration,
// then peak, then index is applied to the staged base and to the candidate's rows.  What bounds a
// step is a chain of LDS latencies (list, walk over the node's edges, range maxima, tables), so
// the workgroup is small and several share a compute unit: 256 threads, 512 where a walker has one to itself
// (queue_merges).  C = 2, up to 32 steps of K = 64 by 256 / 512 / 1024 threads: n = 442, 1024 walkers 168 / 249 / 556 us.  (1024 walkers at n = 442, up to 48 steps: 0.18 ms, 0.25 with one lane per entry, whose edges one
// lane then walks one after the other; 19 with every merge written out as a row of its own and evaluated by
// moc_eval_batch, four launches a step, 9.8 the writing and 7.9 the evaluation.)
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

    // ---- eight lanes per entry (moc_cut_moves.h), the node's inputs and consumers side by side.
    // key = (2^31 - 1 - w_v) << 32 | peak: the lowest duration, then the lowest peak; then the lowest copy index.
    uint64_t best = ~0ull;
    int best_copy = 0x7FFFFFFF;
    const int gl = t & (kGroup - 1);
    for (int r = t / kGroup; r < count; r += NT / kGroup) {
      const int k = list[r];
      const int v = k / C, below = live_below(L.packed, C, k);
      const uint32_t pc = L.packed[k], pb = L.packed[below];
      const uint32_t sc = pc & 0xFFFFu;
      const uint32_t joined = (pb & 0xFFFFu) | (max(pb >> 16, pc >> 16) << 16);
      int vv = gl == 0 ? base_viol : 0;   // shares of the lanes
      // Eq. (3) among the live copies of v, before and after
      int end_before = -1, end_after = -1;
      for (int i = 0; i < C; ++i) {
        const uint32_t p = L.packed[v * C + i];
        if (!live_of(p)) continue;
        const int start = (int)(p & 0xFFFFu);
        vv -= gl == 0 && end_before > start ? 1 : 0;
        end_before = (int)(p >> 16);
        if (v * C + i == k) continue;
        vv += gl == 0 && end_after > start ? 1 : 0;
        end_after = (int)((v * C + i == below ? joined : p) >> 16);
      }
      if (gl == 0 && bit_at(L.occ2, (int)sc)) --vv;   // Eq. (6): a shared start loses one of its copies
      // Eq. (5): the inputs of c are not asked for any more
      for (int x = lists.in_begin(v) + gl, x1 = lists.in_begin(v + 1); x < x1; x += kGroup) {
        const uint32_t* const pu = L.packed + (lists.pair(x) & 0xFFFFu);
        bool held = false;
        for (int i = 0; i < C; ++i) held = held || covers1(pu[i], sc);
        vv -= held ? 0 : 1;
      }
      // Eq. (5): the consumers of v, served by the copies as they stand and as they would be
      for (int y = lists.out_begin(v) + gl, y1 = lists.out_begin(v + 1); y < y1; y += kGroup) {
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
      vv = group_sum(vv);
      if (vv != 0) continue;
      const Range range = merged_range(pc, pb, lists.size_of(v));
      int peak = L.pre[lay.blocks];
      if (range.change != 0) {
        const InOut m = group_range_maxima(L, lay.blocks, range.lo, range.hi, gl);
        peak = max(m.in + range.change, m.out);
      }
      if ((int64_t)peak > g.budget || gl != 0) continue;
      const uint64_t key = (uint64_t)(0x7FFFFFFFu - (uint32_t)g.size_dur[v].y) << 32 | (uint32_t)peak;
      if (key < best || (key == best && k < best_copy)) {
        best = key;
        best_copy = k;
      }
    }
#pragma unroll
    for (int off = kWave / 2; off >= kGroup; off >>= 1) {   // the groups' first lanes
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
    add_ranges<NT, false>(L, lay, &range, 1, 0, T, t);
    if (range.change != 0) build_maxima<NT>(L, lay, t);
  }
  if (t == 0) merges[blockIdx.x] = steps;
}

using DescendKernel = void (*)(GraphView, int32_t*, int32_t*, uint8_t*, int, moc_best_move*, int32_t*, int, MvLayout);

// WIDE: keeping cuts look at all inputs of a node for every stretch between two of the steps they make, and pass
// over the inputs that are held anyway where nodes have more than kWideInputs; the code for it costs other graphs
// 2 % (n = 442, 1024 walkers 550 us, 540 without).  31 nodes of 600 inputs among 620, 64 walkers: 1430 us
// without, 418 with; every 20th of 320 nodes with 300 inputs 211 and 137 (one lane per move: 389, 154).
template <int NT, bool LISTS, int MODE, bool WIDE>
DescendKernel pick_descend(int C) {
  switch (C) {
    case 2: return descend_cuts_kernel<2, NT, LISTS, MODE, WIDE>;
    case 3: return descend_cuts_kernel<3, NT, LISTS, MODE, WIDE>;
    default: return descend_cuts_kernel<0, NT, LISTS, MODE, WIDE>;
  }
}
template <int MODE, bool WIDE>
DescendKernel pick_descend(int C, int nt, bool lists) {
  if (!lists) return pick_descend<1024, false, MODE, WIDE>(C);
  return nt == 256   ? pick_descend<256, true, MODE, WIDE>(C)
         : nt == 512 ? pick_descend<512, true, MODE, WIDE>(C)
                     : pick_descend<1024, true, MODE, WIDE>(C);
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

constexpr int64_t kMaxLaunch = (int64_t)1 << 21;   // candidates per launch: a grid has fewer than 2^32 threads

int queue_cut_descent(const moc_graph* g, int64_t B, int32_t* starts, int32_t* ends, uint8_t* active, int max_steps,
                          int mode, moc_best_move* last_move, int32_t* out_steps, hipStream_t stream) {
  const int T = g->view.T;
  const DescendShape shape = descend_shape(T, g->view.n, g->view.m, B, g->num_cu, g->max_lds);
  const int nt = shape.nt, cap = shape.cap;
  const MvLayout lay = shape.lay;
  if (lay.bytes > g->max_lds) return MOC_EOVERFLOW;
  const bool lists = lay.lists != 0;
  const DescendKernel kern = mode == 0      ? pick_descend<0, false>(g->view.C, nt, lists)
                             : g->view.wide ? pick_descend<1, true>(g->view.C, nt, lists)
                                            : pick_descend<1, false>(g->view.C, nt, lists);
  int per_cu = 0;   // not used: the call is for the kernel's LDS limit
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), nt, lay.bytes, false, &per_cu)) return rc;
  for (int64_t at = 0; at < B; at += kMaxLaunch)
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(B - at, kMaxLaunch)), dim3(nt), lay.bytes, stream, g->view, starts + at * T,
                       ends + at * T, active + at * T, max_steps, last_move + at, out_steps + at, cap, lay);
  return MOC_OK;
}

int queue_merges(const moc_graph* g, int64_t B, int32_t* starts, int32_t* ends, uint8_t* active, int max_steps, int K,
                     int32_t* out_merges, hipStream_t stream) {
  const int T = g->view.T;
  const MvLayout lay = mv_layout(T, g->view.n, g->view.m, (T + 1) / 2, true, g->max_lds);
  if (lay.bytes > g->max_lds) return MOC_EOVERFLOW;
  // One walker to a compute unit: 512 threads, where a base feeds them.  K = 64, 32 to 48 steps, 256 / 512 / 1024 threads: n =
  // 200, 100 walkers 75 / 79 / 97 us; n = 442, 200 walkers 133 / 134 / 160, 500 walkers 143 / 150 / 284; n = 700, 250 walkers 207 / 184 / 208;
  // training graph, n = 1000, 100 walkers 323 / 254 / 291; n = 2000, 100 walkers 534 / 381 / 376.
  const int nt = B <= g->num_cu && T > 900 ? 512 : 256;
  const MergeKernel kern = nt == 512 ? lay.lists ? pick_merge<512, true>(g->view.C) : pick_merge<512, false>(g->view.C)
                                     : lay.lists ? pick_merge<256, true>(g->view.C) : pick_merge<256, false>(g->view.C);
  int per_cu = 0;   // not used: the call is for the kernel's LDS limit
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), nt, lay.bytes, false, &per_cu)) return rc;
  for (int64_t at = 0; at < B; at += kMaxLaunch)
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(B - at, kMaxLaunch)), dim3(nt), lay.bytes, stream, g->view, starts + at * T,
                       ends + at * T, active + at * T, K, max_steps, out_merges + at, lay);
  return MOC_OK;
}

__global__ void fill_zero_kernel(int32_t* p, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace

extern "C" int moc_search_cuts(const moc_graph* g, int64_t B, int32_t* starts, int32_t* ends, uint8_t* active,
                               int32_t max_steps, moc_best_move* work_best, int32_t* out_steps, void* hip_stream) {
  if (!g || B < 0 || max_steps < 0) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (!starts || !ends || !active || !work_best || !out_steps) return MOC_EINVAL;
  if ((((uintptr_t)starts | (uintptr_t)ends | (uintptr_t)out_steps) & 3) || ((uintptr_t)work_best & 7)) return MOC_EINVAL;
  if (B > 0x7FFFFFFFll) return MOC_EINVAL;
  if (const int rc = moc_check_cuts(g)) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (max_steps == 0)
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, stream, out_steps, B);
  else if (const int rc = queue_cut_descent(g, B, starts, ends, active, max_steps, 0, work_best, out_steps, stream))
    return rc;
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

extern "C" int moc_search_two_phase(const moc_graph* g, int64_t B, int32_t* starts, int32_t* ends, uint8_t* active,
                                    int32_t max_cuts, int32_t max_merges, int32_t K, moc_best_move* work_best,
                                    int32_t* work_starts, int32_t* work_ends, uint8_t* work_active,
                                    int32_t* work_list, moc_result* work_results, int32_t* out_cuts,
                                    int32_t* out_merges, void* hip_stream) {
  if (!g || B < 0 || max_cuts < 0 || max_merges < 0 || K < 1) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (!starts || !ends || !active || !work_best || !out_cuts || !out_merges) return MOC_EINVAL;
  if (max_merges > 0 && (!work_starts || !work_ends || !work_active || !work_list || !work_results)) return MOC_EINVAL;
  if ((((uintptr_t)starts | (uintptr_t)ends | (uintptr_t)out_cuts | (uintptr_t)out_merges | (uintptr_t)work_list) & 3) ||
      (((uintptr_t)work_best | (uintptr_t)work_results) & 7))
    return MOC_EINVAL;
  if (((uintptr_t)work_starts | (uintptr_t)work_ends) & 3) return MOC_EINVAL;
  if (B > 0x7FFFFFFFll || (int64_t)B * K > 0x7FFFFFFFll) return MOC_EINVAL;
  if (const int rc = moc_check_cuts(g)) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const unsigned blocks = (unsigned)((B + 255) / 256);
  // Phase 1: towards the budget by cuts that keep the producer's inputs
  if (max_cuts == 0)
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, stream, out_cuts, B);
  else if (const int rc = queue_cut_descent(g, B, starts, ends, active, max_cuts, 1, work_best, out_cuts, stream))
    return rc;
  MOC_HIP(hipGetLastError());
  // Phase 2: undo recomputations while the candidate stays within the budget
  if (max_merges == 0)
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, stream, out_merges, B);
  else if (const int rc = queue_merges(g, B, starts, ends, active, max_merges, K, out_merges, stream))
    return rc;
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}
