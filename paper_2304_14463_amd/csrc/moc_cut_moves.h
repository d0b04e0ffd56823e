// Cut-and-recompute moves of a staged base (see moc_eval_cuts in moccasin.h): which copies and
// positions a move involves, and its score.  For the in-edge (u, v) and a copy of the consumer v
// with start t: copy k of u, the last-starting live copy that covers t, keeps [s_k, last use before
// p]; the lowest inactive copy j of u takes [p, e_k], p a free position in (s_k, t) (mode 0: where
// all inputs of u are held; mode 1: where every input is held or has an earlier copy, which is then
// kept until p).  Every consumer that k covered is covered by one of the two pieces, since no live
// consumer starts in (last use, p], and the new computation finds its inputs by the choice of p.
#pragma once

#include "moc_moves.h"

namespace {

struct Cut {
  int k, j;        // copy of u that is cut, copy of u that becomes active (0 .. C-1)
  int sk, ek;      // interval of copy k as it stands
  int p;           // start of the recomputation
  int last_use;    // new end of copy k
};

// Positions at which the base's profile reaches its peak, countable over any range.
struct PeakCount {
  const uint32_t* bits;
  const int32_t* before;   // per word: such positions in the words below it
  int total;
  __device__ __forceinline__ int within(int lo, int hi) const {   // in [lo, hi], 0 <= lo, hi < T
    const int wl = lo >> 5, wh = hi >> 5;
    const uint32_t bl = bits[wl], bh = bits[wh];
    return before[wh] - before[wl] + (int)__popc(bh & (0xFFFFFFFFu >> (31 - (hi & 31)))) -
           (int)__popc(bl & ((1u << (lo & 31)) - 1u));
  }
};

// Marks the positions at the base's peak.  Ends with a barrier.
template <int NT>
__device__ __forceinline__ PeakCount mark_peak(const BaseLds& L, const MvLayout& lay, int T, int peak, int t) {
  constexpr int NW = NT / kWave;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  for (int c = wave; 2 * c < lay.bit_words; c += NW) {
    const int x = c * kWave + lane;
    const uint64_t hit = __ballot(x < T && L.profile[min(x, T - 1)] == peak);
    if (lane < 2) L.peak_bits[2 * c + lane] = (uint32_t)(hit >> (32 * lane));
  }
  __syncthreads();
  int total = 0;   // every wave counts, the first one writes
  for (int w0 = 0; w0 < lay.bit_words; w0 += kWave) {
    const int w = w0 + lane;
    const int mine = w < lay.bit_words ? (int)__popc(L.peak_bits[w]) : 0;
    const int incl = total + scan_sum(mine);
    if (wave == 0 && w < lay.bit_words) L.peak_before[w] = incl - mine;
    total = last_lane(incl);
  }
  __syncthreads();
  return PeakCount{L.peak_bits, L.peak_before, total};
}

// Is the node whose copies begin at `first` held at position x (a live copy with s < x <= e)?
__device__ __forceinline__ bool held_at(int C, const uint32_t* packed, int first, int x) {
  bool held = false;
  for (int q = 0; q < C; ++q) held = held || covers1(packed[first + q], (uint32_t)x);
  return held;
}

// The largest end below x of a live copy of that node, -1 if none.
__device__ __forceinline__ int latest_end(int C, const uint32_t* packed, int first, int x) {
  int best = -1;
  for (int q = 0; q < C; ++q) {
    const uint32_t p = packed[first + q];
    if (live_of(p) && (int)(p >> 16) < x) best = max(best, (int)(p >> 16));
  }
  return best;
}

// Which copies and positions the move involves; false if it is not applicable.  ub = u*C; `t`: start
// of the (live) consumer copy; clean: the base has no violations -- then every input of u had a
// copy at s_k, so that below t each is held or has an earlier copy, and mode 1 need not look.
// (Loops with the same exit in every lane carry integers, not booleans, to their end.)
template <typename A>
__device__ __forceinline__ bool find_cut(const A& lists, int C, const BaseLds& L, int ub, int t, int mode, bool clean, Cut& cut) {
  const int u = ub / C;
  const int y0 = lists.in_begin(u), y1 = lists.in_begin(u + 1), z0 = lists.out_begin(u), z1 = lists.out_begin(u + 1);
  int k = -1, j = -1, sk = -1, ek = 0;
  for (int q = 0; q < C; ++q) {
    const uint32_t pu = L.packed[ub + q];
    if (covers1(pu, (uint32_t)t) && (int)(pu & 0xFFFFu) > sk) {
      k = q;
      sk = (int)(pu & 0xFFFFu);
      ek = (int)(pu >> 16);
    }
    if (j < 0 && pu == MOC_DEAD) j = q;   // inactive (an active copy that is not well formed is staged otherwise)
  }
  if (k < 0 || j < 0) return false;
  int p = -1;
  for (int hi = t - 1; hi > sk;) {
    // the last free position at or below hi (by words of the start bitmap)
    int pos = -1;
    for (int x = hi; x > sk;) {
      const uint32_t free_bits = ~L.occ1[x >> 5] & (0xFFFFFFFFu >> (31 - (x & 31)));
      if (free_bits) {
        pos = (x & ~31) + 31 - __clz(free_bits);
        break;
      }
      x = (x & ~31) - 1;
    }
    if (pos <= sk) break;
    if (mode == 1) {
      int missing = 0;   // inputs neither held at pos nor with an earlier copy
      if (!clean) {
        for (int y = y0; y < y1; ++y) {
          const int w = (int)(lists.pair(y) & 0xFFFFu);
          missing += held_at(C, L.packed, w, pos) || latest_end(C, L.packed, w, pos) >= 0 ? 0 : 1;
        }
      }
      if (missing == 0) {
        p = pos;
        break;
      }
      hi = pos - 1;
      continue;
    }
    // where an input is missing, the search resumes at the end of that input's nearest earlier copy
    int resume = pos;
    for (int y = y0; y < y1; ++y) {
      const int w = (int)(lists.pair(y) & 0xFFFFu);
      int held = 0, below = -1;
      for (int q = 0; q < C; ++q) {
        const uint32_t pw = L.packed[w + q];
        held |= covers1(pw, (uint32_t)pos) ? 1 : 0;
        if (live_of(pw) && (int)(pw >> 16) < pos) below = max(below, (int)(pw >> 16));
      }
      if (!held) resume = min(resume, below);
    }
    if (resume == pos) {
      p = pos;
      break;
    }
    hi = resume;
  }
  if (p <= sk) return false;
  int last_use = sk;
  for (int y = z0; y < z1; y += 4) {   // four consumers at a time, the last one again beyond the end
    int first[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) first[d] = lists.consumer_copy(min(y + d, z1 - 1), C);
#pragma unroll
    for (int d = 0; d < 4; ++d)
      for (int q = 0; q < C; ++q) {
        const int x = (int)(L.packed[first[d] + q] & 0xFFFFu);   // 0xFFFF (not live) is above every p
        if (x > sk && x < p) last_use = max(last_use, x);
      }
  }
  cut = Cut{k, j, sk, ek, p, last_use};
  return true;
}

// Calls f(w, q, end) for every predecessor of u that is not held at p, w*C first: copy q of it is the
// one the move keeps until p (largest end below p, highest index among equals), `end` its end as it
// stands.  Four predecessors are read at a time.  seen(w): has f been called for w before (a
// predecessor listed several times is kept once: after that it is held).
template <typename A, typename Fn, typename Seen>
__device__ __forceinline__ void for_each_kept_input(const A& lists, int C, const BaseLds& L, int u, int p, Seen seen, Fn f) {
  const int y0 = lists.in_begin(u), y1 = lists.in_begin(u + 1);
  for (int y = y0; y < y1; y += 4) {
    int w[4], best[4], end[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) w[d] = (int)(lists.pair(min(y + d, y1 - 1)) & 0xFFFFu);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      int held = y + d < y1 ? 0 : 1;
      best[d] = -1;
      end[d] = -1;
      for (int q = 0; q < C; ++q) {
        const uint32_t pw = L.packed[w[d] + q];
        held |= covers1(pw, (uint32_t)p) ? 1 : 0;
        if (live_of(pw) && (int)(pw >> 16) < p && (int)(pw >> 16) >= end[d]) {
          best[d] = q;
          end[d] = (int)(pw >> 16);
        }
      }
      if (held) best[d] = -1;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d)
      if (best[d] >= 0 && !seen(w[d], y + d)) f(w[d], best[d], end[d]);
  }
}

struct CutScore { int viol, peak, at; };   // at: positions that still reach the base's peak

// lower_only: moves that raise the peak are of no use and need no score (false as well).
template <typename A>
__device__ __forceinline__ bool score_cut(const A& lists, int C, const BaseLds& L, const MvLayout& lay, int ub, int t, int mode,
                                          int base_viol, int base_peak, const PeakCount& at_peak, bool lower_only,
                                          CutScore& out, Cut& cut) {
  const int blocks = lay.blocks;
  if (!find_cut(lists, C, L, ub, t, mode, base_viol == 0, cut)) return false;
  const int u = ub / C, p = cut.p, last_use = cut.last_use;
  int vv = base_viol;
  // Eq. (3) among the live copies of u, before and after
  int end_before = -1, end_after = -1;
  for (int q = 0; q < C; ++q) {
    const uint32_t pu = L.packed[ub + q];
    if (live_of(pu)) {
      vv -= end_before > (int)(pu & 0xFFFFu) ? 1 : 0;
      end_before = (int)(pu >> 16);
    }
    const uint32_t now = q == cut.k ? (uint32_t)cut.sk | (uint32_t)last_use << 16
                       : q == cut.j ? (uint32_t)p | (uint32_t)cut.ek << 16 : pu;
    if (live_of(now)) {
      vv += end_after > (int)(now & 0xFFFFu) ? 1 : 0;
      end_after = (int)(now >> 16);
    }
  }
  if (cut.j == 0) --vv;   // Eq. (7)
  const int sz = lists.size_of(u);
  int pk = base_peak, at = at_peak.total;
  // mode 1: the inputs that are kept until p.  lo = the lowest position whose memory changes.
  // The first kKept of them are noted (node and end, size) for the walk below, which looks at each
  // of them once per step: finding them again every time costs a pass over the in-edges of u
  // with several reads per edge.
  constexpr int kKept = 8;
  uint32_t kept_end[kKept];   // end + 1, node (times C) << 16
  int kept_size[kKept];
#pragma unroll
  for (int s = 0; s < kKept; ++s) { kept_end[s] = 0; kept_size[s] = 0; }
  int n_kept = 0, lo = last_use + 1;
  // listed before: among those noted, or (more than fit) anywhere earlier in the list
  auto seen = [&](int w, int y) {
    int hit = 0;
    if (n_kept <= kKept) {
#pragma unroll
      for (int s = 0; s < kKept; ++s) hit |= s < n_kept && (int)(kept_end[s] >> 16) == w ? 1 : 0;
    } else {
      for (int z = lists.in_begin(u); z < y; ++z) hit |= (int)(lists.pair(z) & 0xFFFFu) == w ? 1 : 0;
    }
    return hit != 0;
  };
  if (mode == 1)
    for_each_kept_input(lists, C, L, u, p, seen, [&](int w, int q, int end) {
      const int m_w = lists.size_of(w / C);
#pragma unroll
      for (int s = 0; s < kKept; ++s)
        if (s == n_kept) { kept_end[s] = (uint32_t)(end + 1) | (uint32_t)w << 16; kept_size[s] = m_w; }
      ++n_kept;
      lo = min(lo, end + 1);
      // Eq. (3): the kept copy against the next live copy of its node
      int next = -1;
      for (int c = C - 1; c >= 0; --c) {
        const uint32_t nx = L.packed[w + c];
        if (c > q && live_of(nx)) next = (int)(nx & 0xFFFFu);
      }
      if (next >= 0) vv += (p > next ? 1 : 0) - (end > next ? 1 : 0);
      // Eq. (5): consumers of w that start in (end, p] are covered now.  None of them was: a copy
      // of w that covered a position in (end, p] would end at or after p and cover p as well
      // (w would be held there), or end in (end, p), and `end` is the largest end below p.  (So
      // a base without violations has none.)
      if (base_viol != 0) {
        const int wn = w / C;
        for (int y = lists.out_begin(wn), y1 = lists.out_begin(wn + 1); y < y1; ++y) {
          const uint32_t* const px = L.packed + lists.consumer_copy(y, C);
          for (int c = 0; c < C; ++c) {
            const int sx = (int)(px[c] & 0xFFFFu);   // 0xFFFF if not live: above every p
            if (sx > end && sx <= p) --vv;
          }
        }
      }
    });
  if (n_kept == 0) {
    if (last_use + 1 <= p - 1) {
      const InOut m = range_maxima<true>(L, blocks, last_use + 1, p - 1);
      pk = max(m.in - sz, m.out);
      // positions still at the base's peak: those outside the range (all, if nothing is taken away)
      at = pk < base_peak ? 0 : at - (sz > 0 ? at_peak.within(last_use + 1, p - 1) : 0);
    }
  } else {
    // The memory changes on [lo, p]: -m_u on (last_use, p), +m_w on (end_w, p] for every kept
    // input.  All these stretches end at p or just before it, so the change is a step function
    // whose steps are at last_use + 1, at the end_w + 1 and at p: walk it step by step (the next
    // step is found by a pass over the kept inputs; there are few of them).
    int top = range_maxima<true>(L, blocks, lo, p).out;
    int still = at_peak.total - at_peak.within(lo, p);
    for (int from = lo; from <= p;) {
      int next = p + 1, add = 0;   // the step after `from`, and the change on [from, next)
      if (from < last_use + 1) next = min(next, last_use + 1);
      if (from < p) next = min(next, p);
      if (n_kept <= kKept) {
#pragma unroll
        for (int s = 0; s < kKept; ++s) {
          if (s < n_kept) {
            const int begin = (int)(kept_end[s] & 0xFFFFu);
            if (begin > from) next = min(next, begin);
            else add += kept_size[s];
          }
        }
      } else {
        auto listed = [&](int w, int y) {
          int hit = 0;
          for (int z = lists.in_begin(u); z < y; ++z) hit |= (int)(lists.pair(z) & 0xFFFFu) == w ? 1 : 0;
          return hit != 0;
        };
        for_each_kept_input(lists, C, L, u, p, listed, [&](int w, int, int end) {
          if (end + 1 > from) next = min(next, end + 1);
          else add += lists.size_of(w / C);
        });
      }
      if (from >= last_use + 1 && from < p) add -= sz;
      const int here = range_maxima<false>(L, blocks, from, next - 1).in;
      top = max(top, here + add);
      if (lower_only && top > base_peak) return false;
      // positions of [from, next) that reach the base's peak afterwards
      if (add == 0) {
        still += at_peak.within(from, next - 1);
      } else if (add > 0 && here + add >= base_peak) {   // rare: few stretches come near the peak
        still += count_reaching(L, lay, from, next - 1, base_peak - add);
      }
      from = next;
    }
    pk = top;
    at = pk < base_peak ? 0 : still;
  }
  out = CutScore{vv, pk, at};
  return true;
}

// The best of the moves a lane, a wave, a workgroup has seen: lowest (violations, peak, positions
// left at the base's peak, index).
struct BestCut {
  uint64_t score = ~0ull;   // violations << 32 | peak; the scores of real moves stay below
  uint64_t tie = ~0ull;     // positions at the peak << 32 | index
  __device__ __forceinline__ bool take(uint64_t s, uint64_t t) {
    const bool better = s < score || (s == score && t < tie);
    if (better) {
      score = s;
      tie = t;
    }
    return better;
  }
  __device__ __forceinline__ int move() const { return score == ~0ull ? -1 : (int)(uint32_t)tie; }
  __device__ __forceinline__ int viol() const { return (int)(score >> 32); }
  __device__ __forceinline__ int peak() const { return (int)(uint32_t)score; }
  __device__ __forceinline__ int at() const { return (int)(tie >> 32); }
};

// Over the whole workgroup, the same in every thread afterwards.  `words`: 4 per wave, free before
// and after a barrier on either side.
template <int NT>
__device__ __forceinline__ void best_of_workgroup(BestCut& best, int32_t* words, int t) {
  constexpr int NW = NT / kWave;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1)
    best.take((uint64_t)__shfl_xor((unsigned long long)best.score, off), (uint64_t)__shfl_xor((unsigned long long)best.tie, off));
  uint64_t* const slots = reinterpret_cast<uint64_t*>(words);
  if (lane == 0) {
    slots[2 * wave] = best.score;
    slots[2 * wave + 1] = best.tie;
  }
  __syncthreads();
  best = BestCut{};
#pragma unroll
  for (int w = 0; w < NW; ++w) best.take(slots[2 * w], slots[2 * w + 1]);
}

// Scores the moves of the staged base, every wave its share: the moves of 64 in-edges at a time are
// sifted (the consumer's copy live and covered by a copy of the producer), the others get the score
// "not applicable" at once; the survivors wait in a queue of the wave's own and are scored 64 at a
// time, since most moves do not survive and scoring is long.  peak_only (a descent step from a base
// without violations): only moves with a position at the peak inside (s_k, t) -- a move can lower
// the peak or the number of positions that reach it only there.  scored(q, ub, score or none).
template <int CT, int NT, typename A, typename Out>
__device__ __forceinline__ void score_cuts(const GraphView& g, const A& lists, const BaseLds& L, const MvLayout& lay,
                                           int32_t* queue, int mode, int base_viol, int base_peak,
                                           const PeakCount& at_peak, bool peak_only, BestCut& best, int t, Out scored) {
  const int C = CT ? CT : g.C;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  int32_t* const mine = queue + wave * (2 * kWave);
  int queued = 0;
  auto score = [&](int q) {
    const int x = q / C, i = q - x * C;
    const uint32_t pair = lists.pair(x);
    const int ub = (int)(pair & 0xFFFFu);
    const int at = (int)(L.packed[(pair >> 16) + i] & 0xFFFFu);
    CutScore sc;
    Cut cut;
    const bool ok = score_cut(lists, C, L, lay, ub, at, mode, base_viol, base_peak, at_peak, peak_only, sc, cut);
    if (ok) best.take((uint64_t)(uint32_t)sc.viol << 32 | (uint32_t)sc.peak, (uint64_t)(uint32_t)sc.at << 32 | (uint32_t)q);
    scored(q, ub, ok ? &sc : nullptr);
  };
  for (int x0 = wave * kWave; x0 < g.m; x0 += NT) {
    const int x = x0 + lane;
    const uint32_t pair = lists.pair(min(x, g.m - 1));
    for (int i = 0; i < C; ++i) {
      const uint32_t consumer = x < g.m ? L.packed[(pair >> 16) + i] : MOC_DEAD;
      const int at = (int)(consumer & 0xFFFFu);
      int sk = -1;
      if (live_of(consumer))
        for (int c = 0; c < C; ++c) {
          const uint32_t pu = L.packed[(pair & 0xFFFFu) + c];
          if (covers1(pu, (uint32_t)at)) sk = max(sk, (int)(pu & 0xFFFFu));
        }
      bool keep = sk >= 0;
      if (peak_only) {
        int hits = 0;
        if (keep && sk + 1 <= at - 1) hits = at_peak.within(sk + 1, at - 1);
        keep = hits > 0;
      }
      const int q = x * C + i;
      if (!keep && x < g.m) scored(q, 0, nullptr);
      const uint64_t kept = __ballot(keep);
      if (keep) mine[queued + __popcll(kept & ((1ull << lane) - 1))] = q;
      queued += __popcll(kept);
      wave_lds_order();
      if (queued >= kWave) {
        queued -= kWave;
        score(mine[queued + lane]);
        wave_lds_order();
      }
    }
  }
  if (lane < queued) score(mine[lane]);
}

// ---- the best move of a base without violations, without scoring most of the moves
//
// No move of such a base lowers the violations, and none lowers the peak below
//   bound = max(the profile outside (s_k, t), base peak - m_u):
// the memory falls on (last use, p), inside (s_k, t), by m_u, and nowhere else.  So the moves that
// pass the sieve (a position at the peak inside (s_k, t), a copy of u to spare) are noted with their
// bounds, the ones with the lowest bounds are scored first -- as many as fill a wave -- and of the
// others only those whose bound does not exceed the peak reached.  At n = 442 some 200 moves pass
// the sieve and 5 to 50 have to be scored, on the training graph of 1000 nodes 2 of 1000.
struct SiftLds {
  uint32_t* moves;       // [cap] the moves that passed
  uint32_t* where;       // [cap] u*C << 16 | start of the consumer's copy
  uint32_t* bounds;      // [cap] their bounds
  uint16_t* picked;      // [cap] those to be scored next
  uint64_t* node_bits;   // [ceil(n / 64)] bit: a live copy of the node has a position at the peak strictly inside
  int32_t* hist;         // [kBuckets]
  int32_t* counts;       // [0] moves that passed, [1] picked, [2] lowest bound, [3] picked in the second round
  int cap;
};

static_assert(kBuckets == kWave, "one lane per bucket");
__device__ __forceinline__ SiftLds carve_sift(uint32_t* at, int n, int cap) {   // `at`: 8-byte aligned
  SiftLds s;
  s.node_bits = reinterpret_cast<uint64_t*>(at);
  s.moves = at + 2 * ((n + 63) / 64);
  s.where = s.moves + cap;
  s.bounds = s.where + cap;
  s.hist = reinterpret_cast<int32_t*>(s.bounds + cap);
  s.counts = s.hist + kBuckets;
  s.picked = reinterpret_cast<uint16_t*>(s.counts + 4);
  s.cap = cap;
  return s;
}

// True: `best` is the best move over the workgroup and, in the lane that scored it, `cut` the move.
// False: more moves passed than the lists hold, nothing has been scored.  Ends with a barrier.
template <int CT, int NT, typename A>
__device__ __forceinline__ bool best_cut_of_clean_base(const GraphView& g, const A& lists, const BaseLds& L, const MvLayout& lay,
                                                       int32_t* queue, const SiftLds& S, int mode, int base_peak,
                                                       const PeakCount& at_peak, BestCut& best, Cut& cut, bool& mine_is_best, int t) {
  constexpr int NW = NT / kWave;
  const int C = CT ? CT : g.C, n = g.n;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  if (t < kBuckets) S.hist[t] = 0;
  if (t < 4) S.counts[t] = t == 2 ? 0x7FFFFFFF : 0;
  for (int c = wave; c * kWave < n; c += NW) {
    const int v = c * kWave + lane;
    int spans = 0;
    if (v < n)
      for (int i = 0; i < C; ++i) {
        const uint32_t p = L.packed[v * C + i];
        const int s = (int)(p & 0xFFFFu), e = (int)(p >> 16);
        if (live_of(p) && s + 1 <= e - 1) spans += at_peak.within(s + 1, e - 1);
      }
    const uint64_t m = __ballot(spans > 0);
    if (lane == 0) S.node_bits[c] = m;
  }
  __syncthreads();
  // ---- the sieve: in-edges whose producer spans the peak, then 64 of those at a time in full
  int32_t* const mine = queue + wave * (2 * kWave);
  int lowest = 0x7FFFFFFF;
  auto examine = [&](int x, bool have) {
    const uint32_t pair = lists.pair(x);
    const uint32_t* const pu = L.packed + (pair & 0xFFFFu);
    const int u = (int)(pair & 0xFFFFu) / C;
    const int floor_peak = base_peak - lists.size_of(u);
    int spare = 0;
    for (int c = 0; c < C; ++c) spare += pu[c] == MOC_DEAD ? 1 : 0;
    for (int i = 0; i < C; ++i) {
      const uint32_t consumer = have && spare ? L.packed[(pair >> 16) + i] : MOC_DEAD;
      const int at = (int)(consumer & 0xFFFFu);
      int sk = -1, passes = 0;
      if (live_of(consumer))
        for (int c = 0; c < C; ++c)
          if (covers1(pu[c], (uint32_t)at)) sk = max(sk, (int)(pu[c] & 0xFFFFu));
      if (sk >= 0 && sk + 1 <= at - 1) passes = at_peak.within(sk + 1, at - 1);
      const uint64_t m = __ballot(passes > 0);
      if (m == 0) continue;
      int first = 0;
      if (lane == 0) first = atomicAdd(&S.counts[0], (int)__popcll(m));
      first = __builtin_amdgcn_readfirstlane(first);
      const int slot = first + (int)__popcll(m & ((1ull << lane) - 1));
      if (passes > 0 && slot < S.cap) {
        const int bound = max(floor_peak, range_maxima<true>(L, lay.blocks, sk + 1, at - 1).out);
        S.moves[slot] = (uint32_t)(x * C + i);
        S.where[slot] = pair << 16 | (uint32_t)at;
        S.bounds[slot] = (uint32_t)bound;
        lowest = min(lowest, bound);
      }
    }
  };
  int queued = 0;
  for (int x0 = wave * kWave; x0 < g.m; x0 += 4 * NT) {   // four rows of 64 in-edges at a time
    uint32_t u[4];
    uint64_t bits[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) u[d] = (lists.pair(min(x0 + d * NT + lane, g.m - 1)) & 0xFFFFu) / (uint32_t)C;
#pragma unroll
    for (int d = 0; d < 4; ++d) bits[d] = S.node_bits[u[d] >> 6];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int x = x0 + d * NT + lane;
      const int spans = x < g.m ? (int)(bits[d] >> (u[d] & 63)) & 1 : 0;
      const uint64_t kept = __ballot(spans != 0);
      if (spans) mine[queued + __popcll(kept & ((1ull << lane) - 1))] = x;
      queued += __popcll(kept);
      wave_lds_order();
      if (queued >= kWave) {
        queued -= kWave;
        examine(mine[queued + lane], true);
        wave_lds_order();
      }
    }
  }
  if (queued > 0) examine(lane < queued ? mine[lane] : 0, lane < queued);
  atomicMin(&S.counts[2], lowest);
  __syncthreads();
  const int passed = __builtin_amdgcn_readfirstlane(S.counts[0]);
  if (passed > S.cap) {
    __syncthreads();
    return false;
  }
  // ---- how far up the bounds the first round goes: as many whole buckets as fit a wave, at least one
  const int lo_bound = __builtin_amdgcn_readfirstlane(S.counts[2]);
  const float scale = (float)(kBuckets - 1) / (float)max(1, base_peak - lo_bound);
  auto bucket_of = [&](uint32_t bound) { return min(kBuckets - 1, (int)((float)((int)bound - lo_bound) * scale)); };
  int last_bucket = kBuckets - 1;
  if (passed > kWave) {
    for (int r = t; r < passed; r += NT) atomicAdd(&S.hist[bucket_of(S.bounds[r])], 1);
    __syncthreads();
    const int below = scan_sum(S.hist[lane]);
    last_bucket = max((int)__popcll(__ballot(below <= kWave)) - 1, 0);
    if (S.hist[0] > kWave) last_bucket = 0;
  }
  auto pick = [&](int slot_of_count, auto wanted) {   // entries for which `wanted` holds, to `picked`
    for (int r0 = wave * kWave; r0 < passed; r0 += NT) {
      const int r = r0 + lane;
      const bool want = r < passed && wanted(S.bounds[min(r, passed - 1)]);
      const uint64_t m = __ballot(want);
      if (m == 0) continue;
      int first = 0;
      if (lane == 0) first = atomicAdd(&S.counts[slot_of_count], (int)__popcll(m));
      first = __builtin_amdgcn_readfirstlane(first);
      if (want) S.picked[first + (int)__popcll(m & ((1ull << lane) - 1))] = (uint16_t)r;
    }
  };
  BestCut own;
  auto score_picked = [&](int count) {
    for (int r = t; r < count; r += NT) {
      const int at = S.picked[r];
      const uint32_t q = S.moves[at], where = S.where[at];
      CutScore sc;
      Cut c;
      if (score_cut(lists, C, L, lay, (int)(where >> 16), (int)(where & 0xFFFFu), mode, 0, base_peak, at_peak, true, sc, c)) {
        if (own.take((uint64_t)(uint32_t)sc.viol << 32 | (uint32_t)sc.peak, (uint64_t)(uint32_t)sc.at << 32 | q)) cut = c;
      }
    }
  };
  pick(1, [&](uint32_t bound) { return bucket_of(bound) <= last_bucket; });
  __syncthreads();
  const int first_round = __builtin_amdgcn_readfirstlane(S.counts[1]);
  score_picked(first_round);
  best = own;
  best_of_workgroup<NT>(best, L.scratch, t);
  if (first_round < passed) {   // the others, unless their bound lies above what was reached
    const uint64_t reached = best.score;
    pick(3, [&](uint32_t bound) { return bucket_of(bound) > last_bucket && (uint64_t)bound <= reached; });
    __syncthreads();
    const int second_round = __builtin_amdgcn_readfirstlane(S.counts[3]);
    if (second_round > 0) {
      score_picked(second_round);
      best = own;
      best_of_workgroup<NT>(best, L.scratch + 4 * NW, t);
    }
  }
  mine_is_best = own.score == best.score && own.tie == best.tie;
  return true;
}

}  // namespace
