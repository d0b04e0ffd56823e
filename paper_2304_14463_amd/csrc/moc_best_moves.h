// The best single-field move of a base, and the descent by such moves: every move need not be scored for
// that.  (The table of all scores: moc_neighbours_table.hip, where the moves are defined.)
//
// How many violations a move can take away at most is known before any move is scored: an uncovered input can
// be mended by the consumer's start, if a copy of the producer is kept somewhere within R of it, by a move of the
// consumer's that leaves it not live, or by that end of the field of a copy of the producer that lies within R of
// where it is needed; a shared start by its copies, an order pair by its two copies.  One pass over the edges,
// one lane each, counts for each copy and field the violations that its moves could mend (`red`); it counts the
// base's violations on its way.  The fields with the highest count are scored first, one lane per move; what is
// left is scored only if its bound (violations - red, and the base's peak, less the node's size if the field reaches
// over all positions at the peak) is no worse than the best move so far.  Of the 900 to 4000 fields of a schedule 1 to 8
// are scored where it has violations, and about as many as fit one round where it has none; of rows of random intervals,
// whose fields have much the same counts, 1 to 30 (n = 442, 1700 fields), later in a descent 100 to 200.
#pragma once

#include <type_traits>

#include "moc_masks.h"
#include "moc_moves.h"

namespace {

// The moves of one field by a row of 8 or 16 lanes, a displacement each.  What a move changes
// in Eq. (5) sits at few of the node's edges, those whose other end lies within R of the field that moves: each
// lane looks at an edge of its own, and then all of the row take the ones that matter one after the other.
struct MoveScore { int viol, peak; };
struct FieldOf {   // of the row's copy, before the move
  int v, i, field, s, e;
};
template <int CT>
__device__ __forceinline__ MoveScore score_row(const GraphView& g, const BaseLds& L, int blocks, const FieldOf& f, int s2, int e2, int R,
                                               int row_lanes,
                                               int base_viol, int base_peak, int lane) {
  const int T = g.T, C = CT ? CT : g.C, in_row = lane & (row_lanes - 1), row0 = lane & ~(row_lanes - 1);
  const int in_lo = g.in_ptr[f.v], in_hi = g.in_ptr[f.v + 1], out_lo = g.out_ptr[f.v], out_hi = g.out_ptr[f.v + 1];
  const int sz = g.size_dur[f.v].x;
  int u = in_lo + in_row < in_hi ? g.in_idx[in_lo + in_row] : -1;
  int w = out_lo + in_row < out_hi ? g.out_idx[out_lo + in_row] : -1;
  const uint32_t* const row = L.packed + f.v * C;
  const uint32_t before = row[f.i];
  const bool live_old = live_of(before), live_new = (uint32_t)s2 <= (uint32_t)e2 && (uint32_t)e2 < (uint32_t)T;
  const uint32_t after = pack_copy(live_new, s2, e2);
  int d = (live_old ? 1 : 0) - (live_new ? 1 : 0);   // Eq. (2)/(8)
  {   // Eq. (3): each live copy against the next live copy
    int end_old = -1, end_new = -1;
    for (int j = 0; j < C; ++j) {
      const uint32_t p = row[j], q = j == f.i ? after : p;
      if (live_of(p)) {
        d -= end_old > (int)(p & 0xFFFFu) ? 1 : 0;
        end_old = (int)(p >> 16);
      }
      if (live_of(q)) {
        d += end_new > (int)(q & 0xFFFFu) ? 1 : 0;
        end_new = (int)(q >> 16);
      }
    }
  }
  // the row's lanes of `matters`, one after the other; take(lane)
  auto each = [&](lanemask matters, auto take) {
    uint32_t left = (uint32_t)(matters >> row0) & ((1u << row_lanes) - 1);
    while (__any(left != 0)) {
      const int from = row0 + (left ? __ffs(left) - 1 : 0);
      take(from, left != 0);
      left &= left - 1;
    }
  };
  // Eq. (5), the copy as consumer: inputs that are there at some of the starts the field can take and not at others;
  // one that is at none counts as often as the copy is live
  {
    const uint32_t from = (uint32_t)max(f.field == 0 ? f.s - R : f.s, 0), to = (uint32_t)max(f.field == 0 ? f.s + R : f.s, 0);
    const int life = (live_new ? 1 : 0) - (live_old ? 1 : 0);
    for (int x = in_lo; __any(x < in_hi); x += row_lanes) {
      if (x != in_lo) u = x + in_row < in_hi ? g.in_idx[x + in_row] : -1;
      const uint32_t* const inputs = L.packed + max(u, 0) * C;
      const lanemask input = __ballot(u >= 0);
      lanemask always = 0, sometimes = 0;
      for (int j = 0; j < C; ++j) {
        const uint32_t pu = inputs[j];
        always |= spans_lanes(pu, from, to);
        sometimes |= spans_lanes(pu, to, from);
      }
      d += life * __popc((uint32_t)((input & ~sometimes) >> row0) & ((1u << row_lanes) - 1));
      each(input & sometimes & ~always, [&](int lane_of, bool on) {
        const int un = __builtin_amdgcn_ds_bpermute(lane_of << 2, u);
        if (!on) return;
        bool cov_old = !live_old, cov_new = !live_new;
        for (int j = 0; j < C; ++j) {
          const uint32_t pu = L.packed[un * C + j];
          cov_old = cov_old || covers1(pu, (uint32_t)f.s);
          cov_new = cov_new || covers1(pu, (uint32_t)s2);
        }
        d += (cov_old ? 1 : 0) - (cov_new ? 1 : 0);
      });
    }
  }
  // Eq. (5), node v as provider: consumers that no other copy of v covers, at positions the field can reach
  {
    const int from = !live_old || f.field == 0 ? f.s - R : max(f.s, f.e - R);       // below the position
    const int to = !live_old || f.field == 1 ? f.e + R : min(f.s + R, f.e);   // not below it
    for (int x = out_lo; __any(x < out_hi); x += row_lanes) {
      if (x != out_lo) w = x + in_row < out_hi ? g.out_idx[x + in_row] : -1;
      for (int j = 0; j < C; ++j) {
        const uint32_t at = w >= 0 ? L.packed[w * C + j] & 0xFFFFu : 0xFFFFu;
        lanemask held = 0;   // by another copy of v
        for (int q = 0; q < C; ++q) held |= covers_lanes(row[q], at) & __ballot(q != f.i);
        each(low_ne_k(at, 0xFFFFu) & i_gt(at, (uint32_t)from) & ~i_gt(at, (uint32_t)to) & ~held, [&](int lane_of, bool on) {
          const uint32_t t = (uint32_t)__builtin_amdgcn_ds_bpermute(lane_of << 2, (int)at);
          if (on) d += (covers1(before, t) ? 1 : 0) - (covers1(after, t) ? 1 : 0);
        });
      }
    }
  }
  // Eq. (6)
  const bool stays = live_old && live_new && s2 == f.s;
  if (live_old && !stays) d -= bit_at(L.occ2, f.s) ? 1 : 0;
  if (live_new && !stays) d += bit_at(L.occ1, s2) ? 1 : 0;
  // Eq. (4): positions lost or gained
  int lo = 0, hi = -1, change = 0;
  if (live_old && live_new) {
    if (f.field == 0) { lo = min(f.s, s2); hi = max(f.s, s2) - 1; change = s2 < f.s ? sz : -sz; }
    else { lo = min(f.e, e2) + 1; hi = max(f.e, e2); change = e2 > f.e ? sz : -sz; }
  } else if (live_old) { lo = f.s; hi = f.e; change = -sz; }
  else if (live_new) { lo = s2; hi = e2; change = sz; }
  int pk = base_peak;
  if (lo <= hi) {
    const InOut m = range_maxima<true, false>(L, blocks, lo, hi);
    pk = max(max(m.in + change, 0), m.out);
  }
  return MoveScore{base_viol + d, pk};
}

// NT threads, one base at a time.  LOOP: more copies than the threads ask for ahead.  SEARCH: a walker's whole
// descent (its rows stay in LDS and are edited there and in memory alike) instead of one best move.  KEPT: nothing
// writes the rows while the kernel runs.
//
// Bound by the chain of passes over a base, each short and with a barrier behind it: n = 442, 1024 bases, four
// workgroups of 256 to a compute unit, 14 us of a base are 2 staging, 3 the edges, 2 nodes and profile, 2 picking,
// 4.5 scoring in 1.4 rounds.  R = 8, C = 2, n = 442, 1024 bases 43 -> 20 us, n = 1000 72 -> 34, n = 2000, 2048 bases 265 -> 103 (before, one
// lane per copy and field over all that could have fewer violations than the best so far).  Rows of random intervals, where
// few fields can be left out: n = 442, 1024 bases 26 us, 92 while the consumer's start was counted for every uncovered input
// (82 before there were bounds); 256 walkers, 16 steps 411 (770, 520).  80 registers a thread
// with C <= 2, of which a descent spills two (82 are one wave a SIMD fewer: 4096 bases 60 us instead of 51, descents, 3000
// walkers 253 instead of 187, n = 1000, 700 walkers 123 instead of 96; 64 spill, n = 442 26 us), 85 to 92 with more copies,
// five waves; one lane per move with all edges of a node in turn scores in twice the time.
template <bool KEPT>
struct RowPtr { using Ptr = const int32_t* __restrict__; };
template <>
struct RowPtr<false> { using Ptr = const int32_t*; };

struct MoveSteps {
  int32_t *starts, *ends;   // the candidates again, to be edited
  int32_t* steps;           // per candidate: moves applied
  int max_steps;
};

template <int NT, bool LOOP, int CT, bool SEARCH, bool KEPT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(CT == 1 || CT == 2 ? 6 : 5)))
void best_neighbours_kernel(GraphView g, int64_t B, typename RowPtr<KEPT>::Ptr starts,
                                                             typename RowPtr<KEPT>::Ptr ends, const uint8_t* __restrict__ active, int R,
                                                             moc_best_move* __restrict__ out_best, MoveSteps search, BmLayout lay) {
  static_assert(SEARCH != KEPT, "a search edits the rows");
  extern __shared__ uint32_t bm_raw[];
  constexpr int NW = NT / kWave;
  BaseLds L;
  L.carve(bm_raw, lay.base);
  const int blocks = lay.base.blocks;
  uint32_t* const red = bm_raw + lay.red;                                 // per copy: start's count | end's count << 16
  uint16_t* const queue = reinterpret_cast<uint16_t*>(bm_raw + lay.queue);   // copy << 1 | field
  // [0] the base's violations, [1] the highest count, [2], [3] first and last position at the peak, [4..7] fields
  // queued, [8..11] index of the best move of a round (the rounds take turns), [12..13] ~(violations, peak) of the best
  int32_t* const counts = reinterpret_cast<int32_t*>(bm_raw + lay.counts);
  unsigned long long* const reached = reinterpret_cast<unsigned long long*>(bm_raw + lay.counts + 12);
  const int T = g.T, C = CT ? CT : g.C, two_r = 2 * R;
  const int row_lanes = R <= 4 ? 8 : 16, rows = kWave / row_lanes;   // lanes to a field, fields a wave scores at a time
  constexpr uint32_t kMany = 0x7FFF;
  const bool overflows = (int64_t)g.m * C >= kMany - 64;   // more edges than a count can take
  constexpr int kNone = 0x7FFFFFFF;
  constexpr int kFar = 1 << 20;   // beyond T + R, and sums with R stay far from the ends of 32 bits
  constexpr int kEdgesAhead = 6;
  constexpr int kFewRounds = 4;
  const int last_edge = max(g.m - 1, 0);   // (the list of a graph without edges has one entry, too)

  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const int64_t row = b * T;
    int steps = 0;
    for (int step = 0;; ++step) {
      // what derives from the thread index is formed again for every base: kept, it would take registers that the
      // scoring needs
      int t = threadIdx.x;
      asm volatile("" : "+v"(t));
      const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
      if constexpr (SEARCH) {
        if (step >= search.max_steps) break;
      }
      for (int k = t; k < T; k += NT) red[k] = 0;
      if (t < 12) counts[t] = t == 2 || t >= 8 ? kNone : t == 3 ? -1 : 0;
      if (t == 12) *reached = 0;
      uint32_t ahead[kEdgesAhead];   // the first edges: they arrive while the base is staged
#pragma unroll
      for (int d = 0; d < kEdgesAhead; ++d) ahead[d] = g.edge_pair_c[min(d * NT + t, last_edge)];
      // ---- the base: from memory, then (a descent) from the copies in LDS
      int viol = 0;
      if (step == 0) {
        const StageSums sums = stage_copies<CT, NT, LOOP>(g, L, lay.base, starts + row, ends + row, active + row, t);
        viol = sums.viol + sums.live;
      } else {
        for (int x = 4 * t; x < blocks * kBlk; x += 4 * NT) *reinterpret_cast<int4*>(L.profile + x) = make_int4(0, 0, 0, 0);
        for (int w = t; w < lay.base.bit_words; w += NT) { L.occ1[w] = 0; L.occ2[w] = 0; }
        __syncthreads();
        for (int k = t; k < T; k += NT) {
          const uint32_t p = L.packed[k];
          if (k % C == 0 && p == MOC_DEAD) ++viol;        // Eq. (7)
          if (p == (MOC_DEAD | 0x10000u)) ++viol;         // Eq. (2)/(8)
          if (!live_of(p)) continue;
          ++viol;
          const int s = (int)(p & 0xFFFFu), e = (int)(p >> 16), sz = g.size_dur[k / C].x;
          atomicAdd(&L.profile[s], sz);
          if (e + 1 < T) atomicSub(&L.profile[e + 1], sz);
          const uint32_t bit = 1u << (s & 31);
          const uint32_t old = atomicOr(&L.occ1[s >> 5], bit);
          if (old & bit) atomicOr(&L.occ2[s >> 5], bit);
        }
        __syncthreads();
      }
      // ---- violations, and by which fields they could be mended
      constexpr uint32_t kStart = 1, kEnd = 0x10000;
      auto could = [&](int k, uint32_t add) {
        if (overflows) {   // stops about kMany
          const uint32_t now = red[k];
          add &= ((now & 0xFFFFu) < kMany ? kStart : 0u) | (now >> 16 < kMany ? kEnd : 0u);
        }
        if (add != 0) atomicAdd(&red[k], add);
      };
      auto edge = [&](uint32_t pair, lanemask in) {
        const uint32_t* pu = L.packed + (pair & 0xFFFFu);
        const uint32_t* pv = L.packed + (pair >> 16);
        uint32_t copies[CT ? 2 * CT : 1];   // all at once: read one by one they would be read again behind each atomic below
        if constexpr (CT > 0) {
#pragma unroll
          for (int j = 0; j < CT; ++j) { copies[j] = pu[j]; copies[CT + j] = pv[j]; }
          pu = copies;
          pv = copies + CT;
        }
        for (int i = 0; i < C; ++i) {
          const uint32_t copy = pv[i], at = copy & 0xFFFFu;
          lanemask held = 0;
          for (int j = 0; j < C; ++j) held |= covers_lanes(pu[j], at);
          const lanemask miss = low_ne_k(copy, 0xFFFFu) & in & ~held;
          if (miss == 0) continue;
          if (lanes(miss)) {
            const int x = (int)at, until = (int)(copy >> 16);
            ++viol;
            // the consumer not live any more (positions are in [0, T)), or its start where a copy of the producer is kept
            uint32_t mine = until - R < x ? (until < T - 1 ? kStart : 0u) | (x > 0 ? kEnd : 0u) : 0u;
            for (int j = 0; j < C; ++j) {
              const uint32_t p = pu[j];
              const int s = (int)(p & 0xFFFFu), e = (int)(p >> 16);
              const bool close = s - R < x && e + R >= x;   // (no copy that is not live)
              mine |= close && s < e ? kStart : 0u;
              could((int)(pair & 0xFFFFu) + j, close ? (s < x ? kEnd : x > 0 ? kStart : 0u) : p == (MOC_DEAD | 0x10000u) ? kStart | kEnd : 0u);
            }
            could((int)(pair >> 16) + i, mine);
          }
        }
      };
#pragma unroll
      for (int d = 0; d < kEdgesAhead; ++d) {
        const int left = g.m - (d * NT + wave * kWave);   // the same in all lanes
        if (left > 0) edge(ahead[d], left >= kWave ? ~(lanemask)0 : ((lanemask)1 << left) - 1);
      }
      for (int x0 = kEdgesAhead * NT; x0 < g.m; x0 += 4 * NT) {
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
      for (int v = t; v < g.n; v += NT) {
        int prev = -1, end = -1;
        for (int i = 0; i < C; ++i) {
          const int k = v * C + i;
          const uint32_t p = L.packed[k];
          const int s = (int)(p & 0xFFFFu), e = (int)(p >> 16);
          if (!live_of(p)) {
            if (p != MOC_DEAD) could(k, kStart | kEnd);   // Eq. (2)/(8)
            continue;
          }
          if (bit_at(L.occ2, s)) could(k, kStart | (e - R < s && s > 0 ? kEnd : 0u));   // Eq. (6)
          if (end > s) {                                      // Eq. (3)
            ++viol;
            could(prev, kStart | kEnd);
            could(k, kStart | kEnd);
          }
          prev = k;
          end = e;
        }
      }
      for (int w = t; w < lay.base.bit_words; w += NT) viol -= __popc(L.occ1[w]);   // Eq. (6): live copies - distinct starts
      viol = scan_sum(viol);
      if (lane == kWave - 1) atomicAdd(&counts[0], viol);
      scan_profile<NT>(L, lay.base, T, t, [&]() {   // between its two passes: all counts are there
        int top = 0;
        for (int k = t; k < T; k += NT) {
          const uint32_t r = red[k];
          top = max(top, (int)max(r & 0xFFFFu, r >> 16));
        }
        top = scan_max(top);
        if (lane == kWave - 1 && top > 0) atomicMax(&counts[1], top);
      });
      const int base_viol = __builtin_amdgcn_readfirstlane(counts[0]);
      maxima_before_and_from<NT>(L, blocks, t);   // no barrier yet: the first fields can be picked without
      // ---- rounds: fields whose counts lie in [lo, hi), of copies from c0 on, then the next lower counts
      const int top = __builtin_amdgcn_readfirstlane(counts[1]);
      int lo = top - top / 4, hi = top + 1, span = 1, c0 = 0;
      unsigned long long best = 0;   // ~(violations << 32 | peak), 0: none yet
      int best_move = kNone, base_peak = 0;
      bool marked = false;
      for (int round = 0;; ++round) {
        int32_t* const queued = &counts[4 + (round & 3)];
        int32_t* const winner = &counts[8 + (round & 3)];
        if (t == 0) {   // the next round's: last read before the barrier of the round before this
          counts[4 + ((round + 1) & 3)] = 0;
          counts[8 + ((round + 1) & 3)] = kNone;
        }
        const int best_viol = (int)(~best >> 32), best_peak = (int)(uint32_t)~best;   // of no use while best is 0
        const int first = marked ? counts[2] : 0, last = marked ? counts[3] : 0;
        // moves that mend nothing: one round of them mostly has one that leaves the peak where it is
        const bool first_of_many = lo == 0 && (c0 == 0 || best == 0 || best_viol > base_viol || (best_viol == base_viol && best_peak > base_peak));
        int c1 = first_of_many ? min(c0 + NW * rows, T) : T;
        // whether a field that leaves at least `viol` violations can still have the best move
        auto could_win = [&](int k, int f, uint32_t p, int viol, auto with_sizes) {
          if (viol != best_viol) return viol < best_viol;
          const bool earlier = (2 * k + f) * two_r < best_move;
          // only a field that gives up all positions at the peak lowers it, by its node's size at most
          const int s = (int)(p & 0xFFFFu), e = (int)(p >> 16);
          if (live_of(p) && (f == 0 ? s <= first && last < s + R : last <= e && first > e - R)) {
            if (!with_sizes()) return true;
            const int peak = base_peak - g.size_dur[k / C].x;
            return peak < best_peak || (peak == best_peak && earlier);
          }
          return base_peak < best_peak || (base_peak == best_peak && earlier);
        };
        // Where far more are queued than are scored at once: only the upper half of these counts, whose best mostly leaves
        // nothing to do for the others; of a single count those that pass with the sizes of their nodes looked at; no more
        // than there is room for.  Random intervals, n = 442, 256 walkers, 16 steps: 411 us, 1174 with counts taken together as
        // the rounds go on, however many fields that makes.  Every output kept to the end, where all ends lower the peak, R =
        // 8, n = 442, 1024 bases: 23 us, 77 without the sizes (48 before there were bounds).  (They are in memory: looked at
        // for every field, clean rows, n = 442, 3000 walkers, 8 steps take 187 us instead of 182.)
        auto gather = [&](auto with_sizes) {
          for (int k = c0 + t; k < c1; k += NT) {
            const uint32_t p = L.packed[k], r = red[k];
            if (p == MOC_DEAD) continue;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              const int mends = (int)(f == 0 ? r & 0xFFFFu : r >> 16);
              bool take = mends >= lo && mends < hi;
              if (best != 0 && take && mends < (int)kMany) take = could_win(k, f, p, base_viol - mends, with_sizes);
              if (take) {
                const int at = atomicAdd(queued, 1);
                if (at < lay.cap) queue[at] = (uint16_t)(2 * k + f);
              }
            }
          }
          __syncthreads();
          return __builtin_amdgcn_readfirstlane(*queued);
        };
        int count = gather(std::false_type{});
        bool sized = best == 0;
        while (__builtin_expect(count > kFewRounds * NW * rows, 0)) {   // (never more than there is room for)
          if (hi - lo > 1 && c0 == 0 && !overflows) {   // (where counts may have stopped, all that have come first)
            lo = (lo + hi) / 2;
            span = 1;
          } else if (!sized) {
            sized = true;
          } else if (count > lay.cap) {
            c1 = min(c0 + lay.cap / 2, T);
          } else {
            break;
          }
          __syncthreads();
          if (t == 0) *queued = 0;
          __syncthreads();
          count = gather(std::true_type{});
        }
        base_peak = __builtin_amdgcn_readfirstlane(L.pre[blocks]);
        if (count > 0) {
          unsigned long long own = 0;
          int own_move = kNone;
          for (int f0 = wave * rows; f0 < count; f0 += NW * rows) {   // whole waves
            const int at = f0 + (lane >> (31 - __clz(row_lanes)));
            const int entry = queue[min(at, count - 1)], k = entry >> 1, v = k / C;
            const uint32_t p = L.packed[k];
            FieldOf f{v, k - v * C, entry & 1, (int)(p & 0xFFFFu), (int)(p >> 16)};
            if (!live_of(p)) {   // not well formed: its values are not in LDS, and any so far outside the domain do the same
              f.s = min(max(starts[row + k], -kFar), kFar);
              f.e = min(max(ends[row + k], -kFar), kFar);
            }
            for (int d0 = 0; d0 < two_r; d0 += row_lanes) {
              const int disp = d0 + (lane & (row_lanes - 1));
              const int moved = (f.field == 0 ? f.s : f.e) + (disp < R ? disp - R : disp - R + 1);
              const bool applies = at < count && disp < two_r && moved >= 0 && moved < T;
              const MoveScore sc = score_row<CT>(g, L, blocks, f, f.field == 0 && applies ? moved : f.s, f.field == 1 && applies ? moved : f.e, R, row_lanes,
                                                 base_viol, base_peak, lane);
              const unsigned long long key = ~((unsigned long long)(uint32_t)sc.viol << 32 | (uint32_t)sc.peak);
              const int move = entry * two_r + disp;
              if (applies && (key > own || (key == own && move < own_move))) {
                own = key;
                own_move = move;
              }
            }
          }
          if (!marked) {   // positions at the peak
            for (int x = t; x < blocks; x += NT) {
              if (L.table[x] != base_peak) continue;
              for (int j = x * kBlk; j < min((x + 1) * kBlk, T); ++j) {
                if (L.profile[j] != base_peak) continue;
                atomicMin(&counts[2], j);
                atomicMax(&counts[3], j);
              }
            }
            marked = true;
          }
          const unsigned long long most = scan_max64(own);
          if (lane == kWave - 1 && most > best) atomicMax(reached, most);
          __syncthreads();
          const unsigned long long now = *reached;
          if (own != 0 && own == now) atomicMin(winner, own_move);
          __syncthreads();
          best_move = now == best ? min(best_move, *winner) : *winner;
          best = now;
        }
        // ---- what could still be as good
        if (c1 < T) {
          c0 = c1;
          continue;
        }
        c0 = 0;
        hi = lo;
        if (hi <= 0) break;
        if (best != 0) {
          const int best_mends = base_viol - (int)(~best >> 32);
          if (hi - 1 < best_mends) break;
          lo = max(hi - span, best_mends);
        } else {
          lo = hi - span;
        }
        lo = max(lo, hi > 1 ? 1 : 0);   // fields that mend nothing are many, and come by themselves
        span *= 2;
      }
      // ---- the best move; in a descent it is applied if it lowers (violations, max(peak, M), peak)
      moc_best_move r{-1, 0, 0};
      if (best != 0) {
        r.move = best_move;
        r.violations = (int)(~best >> 32);
        r.peak = (int64_t)(uint32_t)~best;
      }
      if (t == 0) out_best[b] = r;
      if constexpr (!SEARCH) break;
      const int64_t m1 = max((int64_t)r.peak, g.budget), m0 = max((int64_t)base_peak, g.budget);
      const bool better = r.move >= 0 && (r.violations < base_viol || (r.violations == base_viol && (m1 < m0 || (m1 == m0 && r.peak < base_peak))));
      if (!better) break;
      ++steps;
      __syncthreads();   // the copies are read no more
      if (t == 0) {
        const int d = r.move % two_r, field = (r.move / two_r) & 1, k = r.move / (2 * two_r);
        int32_t* const at = (field == 0 ? search.starts : search.ends) + row + k;
        const uint32_t p = L.packed[k];
        int s = (int)(p & 0xFFFFu), e = (int)(p >> 16);
        if (!live_of(p)) {
          s = search.starts[row + k];
          e = search.ends[row + k];
        }
        const int moved = (field == 0 ? s : e) + (d < R ? d - R : d - R + 1);
        *at = moved;
        (field == 0 ? s : e) = moved;
        L.packed[k] = (uint32_t)s <= (uint32_t)e && (uint32_t)e < (uint32_t)T ? (uint32_t)s | (uint32_t)e << 16 : MOC_DEAD | 0x10000u;
      }
      __syncthreads();
    }
    if constexpr (SEARCH) {
      if (threadIdx.x == 0) search.steps[b] = steps;
    }
    __syncthreads();
  }
}

}  // namespace
