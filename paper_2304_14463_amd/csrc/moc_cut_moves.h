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
  const int32_t* before;   // per word: such positions in the words below it (set where there are two or more)
  int total, first, last;
  __device__ __forceinline__ int within(int lo, int hi) const {   // in [lo, hi], 0 <= lo, hi < T
    if (total == 1) return lo <= first && first <= hi ? 1 : 0;   // the same in all lanes, and most often so
    const int wl = lo >> 5, wh = hi >> 5;
    const uint32_t bl = bits[wl], bh = bits[wh];
    return before[wh] - before[wl] + (int)__popc(bh & (0xFFFFFFFFu >> (31 - (hi & 31)))) -
           (int)__popc(bl & ((1u << (lo & 31)) - 1u));
  }
  // Is there one strictly between lo and hi?  (0 or 1; two positions settle it unless both lie outside on
  // either side and there are others between them.)
  __device__ __forceinline__ int between(int lo, int hi) const {
    int found = lo < first && first < hi ? 1 : 0;
    if (total > 1) {   // the same in all lanes
      found |= lo < last && last < hi ? 1 : 0;
      if (total > 2 && !found && first <= lo && last >= hi && lo + 1 <= hi - 1) found = within(lo + 1, hi - 1) > 0 ? 1 : 0;
    }
    return found;
  }
};

// The marks as add_ranges left them (behind a barrier).  Ends with a barrier where there are several.
template <int NT>
__device__ __forceinline__ PeakCount count_marks(const BaseLds& L, const MvLayout& lay, int t) {
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  PeakCount c{L.peak_bits, L.peak_before, __builtin_amdgcn_readfirstlane(L.marks[0]),
              __builtin_amdgcn_readfirstlane(L.marks[1]), __builtin_amdgcn_readfirstlane(L.marks[2])};
  if (c.total > 1) {
    if (wave == 0) {
      int before = 0;
      for (int w0 = 0; w0 < lay.bit_words; w0 += kWave) {
        const int w = w0 + lane;
        const int mine = w < lay.bit_words ? (int)__popc(L.peak_bits[w]) : 0;
        const int incl = before + scan_sum(mine);
        if (w < lay.bit_words) L.peak_before[w] = incl - mine;
        before = last_lane(incl);
      }
    }
    __syncthreads();
  }
  return c;
}

// Marks the positions at the base's peak (clear_marks before, a barrier between).  Ends with a barrier.
template <int NT>
__device__ __forceinline__ PeakCount mark_peak(const BaseLds& L, const MvLayout& lay, int T, int peak, int t) {
  constexpr int NW = NT / kWave;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  for (int c = wave; 2 * c < lay.bit_words; c += NW) {
    const int x = c * kWave + lane;
    const uint64_t hit = __ballot(x < T && L.profile[min(x, T - 1)] == peak);
    if (lane < 2) L.peak_bits[2 * c + lane] = (uint32_t)(hit >> (32 * lane));
    if (hit != 0 && lane == 0) {
      atomicAdd(&L.marks[0], (int)__popcll(hit));
      atomicMin(&L.marks[1], c * kWave + (int)__ffsll((unsigned long long)hit) - 1);
      atomicMax(&L.marks[2], c * kWave + 63 - (int)__clzll((long long)hit));
    }
  }
  __syncthreads();
  return count_marks<NT>(L, lay, t);
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

// The last free position in (sk, hi], at or below sk if there is none (by words of the start bitmap).
__device__ __forceinline__ int last_free(const BaseLds& L, int sk, int hi) {
  int pos = -1;
  for (int x = hi; x > sk;) {
    const uint32_t free_bits = ~L.occ1[x >> 5] & (0xFFFFFFFFu >> (31 - (x & 31)));
    if (free_bits) {
      pos = (x & ~31) + 31 - __clz(free_bits);
      break;
    }
    x = (x & ~31) - 1;
  }
  return pos;
}

// The last start in (sk, p) of the consumers z0 .. z1 - 1, sk if there is none.
template <typename A>
__device__ __forceinline__ int last_use_before(const A& lists, int C, const BaseLds& L, int z0, int z1, int sk, int p) {
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
  return last_use;
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
    const int pos = last_free(L, sk, hi);
    if (pos <= sk) break;
    if (mode == 1) {
      int missing = 0;   // inputs neither held at pos nor with an earlier copy
      if (!clean) {
        for (int y = y0; y < y1; ++y) {
          const int w = (int)(lists.pair(y) & 0xFFFFu);
          missing += held_at(C, L.packed, w, pos) || latest_end(C, L.packed, w, pos) >= 0 ? 0 : 1;
        }
      }
      // An input that is missing at pos is missing below it, too: none of its live copies ends before pos or covers it,
      // so all of them start at pos or behind it.  The last free position decides.  (Going on to the next one down until
      // s_k: tables of keeping cuts, half of the bases with violations, n = 1000, 256 bases, C = 2
      // 666 -> 135 us, C = 4 3172 -> 232; n = 2000, C = 3, 100 bases 2593 -> 236.)
      if (missing == 0) p = pos;
      break;
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
  cut = Cut{k, j, sk, ek, p, last_use_before(lists, C, L, z0, z1, sk, p)};
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
// NEAREST: the smallest distance of two lanes that hold something.
template <int NT, int NEAREST = 1>
__device__ __forceinline__ void best_of_workgroup(BestCut& best, int32_t* words, int t) {
  constexpr int NW = NT / kWave;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
#pragma unroll
  for (int off = kWave / 2; off >= NEAREST; off >>= 1)
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
      int kept_one = sk >= 0 ? 1 : 0;
      if (peak_only && kept_one) kept_one = at_peak.between(sk, at);
      const bool keep = kept_one != 0;
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
// No move of such a base lowers the violations, one that raises them is of no use, and none lowers the peak
// below
//   bound = max(the profile's whole blocks outside (s_k, t), base peak - m_u):
// the memory falls on (last use, p), inside (s_k, t), by m_u, and nowhere else.  So the moves that
// pass the sieve (a position at the peak inside (s_k, t), a copy of u to spare) are noted with their
// bounds, the ones with the lowest bounds are scored first, and of the others only those whose bound does
// not exceed the peak reached.  For cuts that keep inputs the bound takes in the place of the computation, the
// last use before it and the inputs carried across the peak.  n = 442: 170 to 190 moves pass the sieve, 26 are
// scored (80 to 120 without the inputs in the bound); training graph of 1000 nodes: 900 and 29.
//
// Eight lanes score a move: the lists of a node's inputs and consumers and the blocks at the ends of a range
// of positions are taken by the lanes side by side, and every stretch of the profile that a move changes
// has a lane of its own.  One lane per move left 3 waves of 4 (15 of 16) idle through a chain of dependent
// reads: n = 442, cuts that keep inputs, 12 to 15 us a step, now 3.3; n = 1000, plain cuts, 3.7, now 1.3.  (Plain cuts
// of which there are many go by lanes all the same where workgroups share a compute unit: kByLanes below.)
struct SiftLds {
  uint32_t* moves;       // [cap] the moves that passed
  uint32_t* where;       // [cap] u*C << 16 | start of the consumer's copy
  uint32_t* bounds;      // [cap] their bounds
  uint16_t* picked;      // [cap] those to be scored next
  int32_t* hist;         // [kBuckets]
  int32_t* counts;       // [0] moves that passed, [1] picked, [2] lowest bound, [3] picked in the second round
  int cap;
};

// Lanes that score a move (four: n = 442, 1024 walkers, two phases 802 us instead of 758 and, on other inputs, 1259
// instead of 1184; on the first kernel with groups), and moves that are scored before the bounds of the others are
// looked at.  With 16 / 32 / 64 of them, several walkers to a compute unit: keeping cuts, n = 442, 1024 walkers 537 /
// 542 / 567 us, plain cuts, training graph, n = 1000, 1024 walkers 660 / 651 / 681.  One walker to a compute unit, whose
// 128 groups take more at once: keeping cuts, n = 442, 32 walkers 410 / 405 / 390; plain cuts, n = 1000, 32 walkers 565 /
// 504 / 443, training graph 275 / 277 / 278; with 32 / 64 / 128, out-degrees falling as 200 / rank^0.7, n = 1903, 97
// walkers, 1460 / 729 / 377, n = 737, 72 walkers 236 / 79 / 75, but the training graph 277 / 278 / 292.
constexpr int kGroup = 8;
constexpr int first_round_moves(int nt) { return nt == 1024 ? 64 : 32; }
// A producer with more consumers than this has a move for each, and each of them would walk them all for its bound:
// it gets the one of plain cuts (C = 5, n = 1600, out-degrees falling as 200 / rank^0.7, 53 walkers, 24 steps, by 16 /
// 32 / 64 / no limit 1155 / 1382 / 1936 / 4541 us; 30 consumers a node, n = 600, 32 walkers 6270 / 2008 / 2067 / 2011).
constexpr int kLongList = 32;
constexpr int kNoBound = 0x7FFFFFFF;   // of a move that is of no use

static_assert(kBuckets == kWave, "one lane per bucket");
__device__ __forceinline__ SiftLds carve_sift(uint32_t* at, int cap) {
  SiftLds s;
  s.moves = at;
  s.where = s.moves + cap;
  s.bounds = s.where + cap;
  s.hist = reinterpret_cast<int32_t*>(s.bounds + cap);
  s.counts = s.hist + kBuckets;
  s.picked = reinterpret_cast<uint16_t*>(s.counts + 4);
  s.cap = cap;
  return s;
}

// Eight consecutive lanes.  All of them are switched on or none is, so that the lane shifts below
// always find their partner.
template <int K>
__device__ __forceinline__ int group_xor(int x) {   // the value of lane ^ K
  constexpr int kQuad[4] = {0, 0xB1, 0x4E, 0x1B};   // quad_perm: lane ^ 1, 2, 3
  if constexpr (K >= 4) x = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true);   // row_half_mirror: lane ^ 7
  constexpr int kRest = K >= 4 ? K ^ 7 : K;
  if constexpr (kRest != 0) x = __builtin_amdgcn_update_dpp(0, x, kQuad[kRest], 0xF, 0xF, true);
  return x;
}
__device__ __forceinline__ int group_max(int x) {
  x = max(x, group_xor<1>(x));
  x = max(x, group_xor<2>(x));
  return max(x, group_xor<7>(x));
}
__device__ __forceinline__ int group_min(int x) {
  x = min(x, group_xor<1>(x));
  x = min(x, group_xor<2>(x));
  return min(x, group_xor<7>(x));
}
__device__ __forceinline__ int group_sum(int x) {
  x += group_xor<1>(x);
  x += group_xor<2>(x);
  return x + group_xor<7>(x);
}

// Maxima of the profile over [lo, hi] and over all other positions, by a group (gl: the lane in it).
__device__ __forceinline__ InOut group_range_maxima(const BaseLds& L, int blocks, int lo, int hi, int gl) {
  const int bl = lo / kBlk, bh = hi / kBlk;
  const int first = bl + 1, count = bh - first;   // whole blocks between
  InOut r{0, max(L.pre[bl], L.suf[bh + 1])};
  if (count > 0) r.in = blocks_maximum(L, blocks, first, count);
  static_assert(kBlk == kGroup, "a position of the blocks at either end per lane");
  const int xl = bl * kBlk + gl, xh = bh * kBlk + gl;
  const int vl = L.profile[xl], vh = L.profile[xh];
  const bool in_l = lo <= xl && xl <= hi, in_h = lo <= xh && xh <= hi;
  r.in = group_max(max(r.in, max(in_l ? vl : 0, in_h ? vh : 0)));
  r.out = group_max(max(r.out, max(in_l ? 0 : vl, in_h ? 0 : vh)));
  return r;
}

// score_cut for a base without violations, by a group: false also for a move that raises the violations or
// the peak.  It says for such a base what find_cut and score_cut say for any: a change to the rule of the move has to
// be made in both.  WIDE: for graphs with nodes of many inputs.  (Loops that groups leave at different times carry integers, not booleans, to their end.)
template <int MODE, bool WIDE, typename A>
__device__ __forceinline__ bool score_cut_by_group(const A& lists, int C, bool parallel, const BaseLds& L, const MvLayout& lay,
                                                   int ub, int t, int base_peak, const PeakCount& at_peak, CutScore& out,
                                                   Cut& cut, int gl) {
  const int blocks = lay.blocks, u = ub / C;
  const int y0 = lists.in_begin(u), y1 = lists.in_begin(u + 1), z0 = lists.out_begin(u), z1 = lists.out_begin(u + 1);
  const int sz = lists.size_of(u);
  int k = -1, j = -1, sk = -1, ek = 0;
  for (int q = 0; q < C; ++q) {
    const uint32_t pu = L.packed[ub + q];
    if (covers1(pu, (uint32_t)t) && (int)(pu & 0xFFFFu) > sk) {
      k = q;
      sk = (int)(pu & 0xFFFFu);
      ek = (int)(pu >> 16);
    }
    if (j < 0 && pu == MOC_DEAD) j = q;
  }
  if (k < 0 || j < 0) return false;
  // ---- where the computation goes (find_cut)
  int p = -1;
  for (int hi = t - 1; hi > sk;) {
    const int pos = last_free(L, sk, hi);
    if (pos <= sk) break;
    int resume = pos;   // mode 1: every input had a copy at s_k, so that each is held or has an earlier one
    if (MODE == 0) {
      for (int y = y0 + gl; y < y1; y += kGroup) {
        const int w = (int)(lists.pair(y) & 0xFFFFu);
        int held = 0, below = -1;
        for (int q = 0; q < C; ++q) {
          const uint32_t pw = L.packed[w + q];
          held |= covers1(pw, (uint32_t)pos) ? 1 : 0;
          if (live_of(pw) && (int)(pw >> 16) < pos) below = max(below, (int)(pw >> 16));
        }
        if (!held) resume = min(resume, below);
      }
      resume = group_min(resume);
    }
    if (resume == pos) {
      p = pos;
      break;
    }
    hi = resume;
  }
  if (p <= sk) return false;
  int last_use = sk;
  for (int z = z0 + gl; z < z1; z += kGroup) {
    const uint32_t* const pc = L.packed + lists.consumer_copy(z, C);
    for (int q = 0; q < C; ++q) {
      const int x = (int)(pc[q] & 0xFFFFu);   // 0xFFFF (not live) is above every p
      if (x > sk && x < p) last_use = max(last_use, x);
    }
  }
  last_use = group_max(last_use);
  cut = Cut{k, j, sk, ek, p, last_use};
  // Eq. (3) among the live copies of u afterwards
  int vv = 0, end_after = -1;
  for (int q = 0; q < C; ++q) {
    const uint32_t pu = L.packed[ub + q];
    const uint32_t now = q == k ? (uint32_t)sk | (uint32_t)last_use << 16 : q == j ? (uint32_t)p | (uint32_t)ek << 16 : pu;
    if (live_of(now)) {
      vv += end_after > (int)(now & 0xFFFFu) ? 1 : 0;
      end_after = (int)(now >> 16);
    }
  }
  if (vv != 0) return false;

  if (MODE == 0) {
    int pk = base_peak, at = at_peak.total;
    if (last_use + 1 <= p - 1) {
      const InOut m = group_range_maxima(L, blocks, last_use + 1, p - 1, gl);
      pk = max(m.in - sz, m.out);
      at = pk < base_peak ? 0 : at - (sz > 0 ? at_peak.within(last_use + 1, p - 1) : 0);
    }
    out = CutScore{0, pk, at};
    return true;
  }
  // ---- the inputs that are kept until p.  The memory changes by a step function: -m_u from last_use + 1 until
  // p - 1 and +m_w from end_w + 1 until p for every kept input.  Step 0 is u's, step i input y0 + i - 1's; a lane
  // looks after every eighth step and the stretch from it to the next one.
  constexpr int kNone = 0x7FFFFFFF;
  struct Step { int begin, size; };
  const int n_steps = 1 + y1 - y0;
  auto step_of = [&](int i, int& order) -> Step {
    if (i == 0) return last_use + 1 < p ? Step{last_use + 1, -sz} : Step{kNone, 0};
    if (i >= n_steps) return Step{kNone, 0};
    const int y = y0 + i - 1, w = (int)(lists.pair(y) & 0xFFFFu);
    int held = 0, kept = -1, end = -1, next = -1;
    for (int q = 0; q < C; ++q) {
      const uint32_t pw = L.packed[w + q];
      held |= covers1(pw, (uint32_t)p) ? 1 : 0;
      if (live_of(pw) && (int)(pw >> 16) < p && (int)(pw >> 16) >= end) {
        kept = q;
        end = (int)(pw >> 16);
      }
    }
    if (held || kept < 0) return Step{kNone, 0};
    if (parallel) {   // listed before: it is kept already
      for (int z = y0; z < y; ++z) held |= (int)(lists.pair(z) & 0xFFFFu) == w ? 1 : 0;
      if (held) return Step{kNone, 0};
    }
    for (int q = C - 1; q >= 0; --q) {   // Eq. (3): the kept copy against the next live copy of its node
      const uint32_t pw = L.packed[w + q];
      if (q > kept && live_of(pw)) next = (int)(pw & 0xFFFFu);
    }
    if (next >= 0 && p > next) order = 1;
    return Step{end + 1, lists.size_of(w / C)};
  };
  // WIDE: which eights of steps hold any (a bit for each, for several of them from 33 eights on); most inputs of a
  // node with many are held.
  uint32_t eights = 0;
  const int per_bit = max(0, 27 - __clz((n_steps - 1) / kGroup));
  const auto bit_of = [&](int i0) { return (uint32_t)i0 / kGroup >> per_bit; };
  const auto empty = [&](int i0) { return WIDE && (eights >> bit_of(i0) & 1) == 0; };
  // f(begin, end, change, first): the stretch behind a step; first: no earlier step begins there
  auto stretches = [&](auto f) {
    for (int i0 = 0; i0 < n_steps; i0 += kGroup) {
      if (empty(i0)) continue;   // the same in all lanes of the group
      int ignored = 0;
      const Step own = step_of(i0 + gl, ignored);
      int next = p, change = own.size, first = 1;
      for (int o0 = 0; o0 < n_steps; o0 += kGroup) {
        if (empty(o0)) continue;
        const Step o = o0 == i0 ? own : step_of(o0 + gl, ignored);
        auto meet = [&](int begin, int size, int index) {
          if (begin > own.begin) next = min(next, begin);
          else change += size;
          if (begin == own.begin && index < i0 + gl) first = 0;
        };
        if (o0 != i0) meet(o.begin, o.size, o0 + gl);
        meet(group_xor<1>(o.begin), group_xor<1>(o.size), o0 + (gl ^ 1));
        meet(group_xor<2>(o.begin), group_xor<2>(o.size), o0 + (gl ^ 2));
        meet(group_xor<3>(o.begin), group_xor<3>(o.size), o0 + (gl ^ 3));
        meet(group_xor<4>(o.begin), group_xor<4>(o.size), o0 + (gl ^ 4));
        meet(group_xor<5>(o.begin), group_xor<5>(o.size), o0 + (gl ^ 5));
        meet(group_xor<6>(o.begin), group_xor<6>(o.size), o0 + (gl ^ 6));
        meet(group_xor<7>(o.begin), group_xor<7>(o.size), o0 + (gl ^ 7));
      }
      if (own.begin < next) f(own.begin, next - 1, change, first);   // (kNone: above every end)
    }
  };
  int lo = p, kept_size = 0, order = 0;
  for (int i0 = 0; i0 < n_steps; i0 += kGroup) {
    const Step own = step_of(i0 + gl, order);
    lo = min(lo, own.begin);
    kept_size += i0 + gl == 0 ? 0 : own.size;
    if (WIDE) eights |= (own.begin != kNone ? 1u : 0u) << bit_of(i0);
  }
  if (WIDE) {
    eights |= (uint32_t)group_xor<1>((int)eights);
    eights |= (uint32_t)group_xor<2>((int)eights);
    eights |= (uint32_t)group_xor<7>((int)eights);
  }
  if (group_max(order) != 0) return false;
  lo = group_min(lo);
  kept_size = group_sum(kept_size);
  const int at_p = L.profile[p];
  int top = max(group_range_maxima(L, blocks, lo, p, gl).out, at_p + kept_size);
  stretches([&](int begin, int end, int change, int) { top = max(top, range_maxima<false>(L, blocks, begin, end).in + change); });
  top = group_max(top);
  if (top > base_peak) return false;
  int still = 0;
  if (top == base_peak) {   // positions that reach the base's peak afterwards
    int here = 0;
    stretches([&](int begin, int end, int change, int first) {
      if (!first) return;
      if (change == 0) here += at_peak.within(begin, end);
      else if (change > 0) here += count_reaching(L, lay, begin, end, base_peak - change);
    });
    still = at_peak.total - at_peak.within(lo, p) + group_sum(here) +
            (kept_size == 0 ? at_peak.within(p, p) : at_p + kept_size >= base_peak ? 1 : 0);
  }
  out = CutScore{0, top, still};
  return true;
}

// True: `best` is the best move over the workgroup and, in the lane that scored it, `cut` the move.
// False: more moves passed than the lists hold, nothing has been scored.  Ends with a barrier.
template <int CT, int NT, int MODE, bool WIDE, typename A>
__device__ __forceinline__ bool best_cut_of_clean_base(const GraphView& g, const A& lists, const BaseLds& L, const MvLayout& lay,
                                                       const SiftLds& S, int base_peak, const PeakCount& at_peak,
                                                       BestCut& best, Cut& cut, bool& mine_is_best, int t) {
  constexpr int NW = NT / kWave;
  const int C = CT ? CT : g.C;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  // ---- the sieve, one lane per in-edge, one copy of the consumer after the other.  (The in-edges whose producer
  // spans a position at the peak first, in a queue per wave, and then 64 of those at a time: n = 442, 1024
  // walkers 611 us instead of 606, n = 1000, 32 walkers 313 instead of 275.)
  int lowest = kNoBound;
  auto note_bound = [&](int r, int u, int lo, int hi, int carried) {   // the memory falls on (lo, hi) at most
    const int outside = max(L.pre[(lo + 1) / kBlk], L.suf[(hi - 1) / kBlk + 1]);
    const int bound = max(base_peak - lists.size_of(u) + carried, outside);
    S.bounds[r] = (uint32_t)(bound <= base_peak ? bound : kNoBound);
    if (bound <= base_peak) lowest = min(lowest, bound);
  };
  for (int x0 = wave * kWave; x0 < g.m; x0 += NT) {
    const int x = min(x0 + lane, g.m - 1), have = x0 + lane < g.m ? 1 : 0;
    const uint32_t pair = lists.pair(x);
    const uint32_t* const pu = L.packed + (pair & 0xFFFFu);
    int spare = 0;
    for (int c = 0; c < C; ++c) spare += pu[c] == MOC_DEAD ? have : 0;
    for (int i = 0; i < C; ++i) {
      const int at = (int)(L.packed[(pair >> 16) + i] & 0xFFFFu);   // 0xFFFF: not live, covered by nothing
      if (__ballot(at != 0xFFFF && at > at_peak.first && spare > 0) == 0) continue;   // most further copies are not live
      int sk = -1, passes = 0;
      for (int c = 0; c < C; ++c)
        if (at != 0xFFFF && covers1(pu[c], (uint32_t)at)) sk = max(sk, (int)(pu[c] & 0xFFFFu));
      if (sk >= 0 && spare > 0) passes = at_peak.between(sk, at);
      const uint64_t m = __ballot(passes != 0);
      if (m == 0) continue;
      int first = 0;
      if (lane == 0) first = atomicAdd(&S.counts[0], (int)__popcll(m));
      first = __builtin_amdgcn_readfirstlane(first);
      const int slot = first + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (passes && slot < S.cap) {
        S.moves[slot] = (uint32_t)(x * C + i);
        S.where[slot] = pair << 16 | (uint32_t)at;
        if (MODE == 0) note_bound(slot, (int)(pair & 0xFFFFu) / C, sk, at, 0);
      }
    }
  }
  if (MODE == 1) __syncthreads();
  const int passed_mode1 = MODE == 1 ? __builtin_amdgcn_readfirstlane(S.counts[0]) : 0;
  // Cuts that keep inputs find their place p without asking for the inputs, so that p and the last use before it
  // are at hand: the memory falls between these two only, and a move without a position at the peak there
  // is of no use.  (The others may go further down for the inputs' sake.)  At such a position, what the inputs
  // add that have to be carried across it is known as well; most moves come to nothing by that.
  if (MODE == 1 && passed_mode1 <= S.cap) {
    for (int r = t; r < passed_mode1; r += NT) {
      const uint32_t where = S.where[r];
      const int ub = (int)(where >> 16), at = (int)(where & 0xFFFFu), u = ub / C;
      const int z0 = lists.out_begin(u), z1 = lists.out_begin(u + 1);
      int sk = -1;
      for (int c = 0; c < C; ++c) {
        const uint32_t pu = L.packed[ub + c];
        if (covers1(pu, (uint32_t)at)) sk = max(sk, (int)(pu & 0xFFFFu));
      }
      if (z1 - z0 > kLongList) {
        note_bound(r, u, sk, at, 0);
        continue;
      }
      const int p = last_free(L, sk, at - 1);
      int last = sk, useful = 0;
      if (p > sk) {
        last = last_use_before(lists, C, L, z0, z1, sk, p);
        useful = at_peak.between(last, p);
      }
      S.bounds[r] = (uint32_t)kNoBound;
      if (useful) {
        const int x = last < at_peak.first && at_peak.first < p ? at_peak.first : last < at_peak.last && at_peak.last < p ? at_peak.last : -1;
        int carried = 0;
        if (g.parallel == 0)   // (an input listed twice is carried once; left as soon as the move raises the peak)
          for (int y = lists.in_begin(u), y1 = lists.in_begin(u + 1); y < y1 && carried <= lists.size_of(u); y += 4) {   // four at a time, the last one again beyond the end
            int w[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) w[d] = (int)(lists.pair(min(y + d, y1 - 1)) & 0xFFFFu);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              int held = y + d < y1 ? 0 : 1, end = -1;
              for (int c = 0; c < C; ++c) {
                const uint32_t pw = L.packed[w[d] + c];
                held |= covers1(pw, (uint32_t)p) ? 1 : 0;
                if (live_of(pw) && (int)(pw >> 16) < p) end = max(end, (int)(pw >> 16));
              }
              if (!held && end < x) carried += lists.size_of(w[d] / C);
            }
          }
        note_bound(r, u, last, p, carried);
      }
    }
  }
  lowest = kNoBound - last_lane(scan_max(kNoBound - lowest));
  if (lane == 0) atomicMin(&S.counts[2], lowest);
  __syncthreads();
  const int passed = __builtin_amdgcn_readfirstlane(S.counts[0]);
  if (passed > S.cap) {
    __syncthreads();
    return false;
  }
  // ---- how far up the bounds the first round goes: as many whole buckets as the groups take at once, at least one
  const int lo_bound = __builtin_amdgcn_readfirstlane(S.counts[2]);
  const float scale = (float)(kBuckets - 1) / (float)max(1, base_peak - lo_bound);
  auto bucket_of = [&](uint32_t bound) { return min(kBuckets - 1, (int)((float)((int)bound - lo_bound) * scale)); };
  int last_bucket = kBuckets - 1;
  if (passed > first_round_moves(NT)) {
    for (int r = t; r < passed; r += NT)
      if (S.bounds[r] != (uint32_t)kNoBound) atomicAdd(&S.hist[bucket_of(S.bounds[r])], 1);
    __syncthreads();
    const int below = scan_sum(S.hist[lane]);
    last_bucket = max((int)__popcll(__ballot(below <= first_round_moves(NT))) - 1, 0);
    if (S.hist[0] > first_round_moves(NT)) last_bucket = 0;
  }
  auto pick = [&](int slot_of_count, auto wanted) {   // entries for which `wanted` holds, to `picked`
    for (int r0 = wave * kWave; r0 < passed; r0 += NT) {
      const int r = r0 + lane;
      const uint32_t bound = S.bounds[min(r, max(passed - 1, 0))];
      const bool want = r < passed && bound != (uint32_t)kNoBound && wanted(bound);
      const uint64_t m = __ballot(want);
      if (m == 0) continue;
      int first = 0;
      if (lane == 0) first = atomicAdd(&S.counts[slot_of_count], (int)__popcll(m));
      first = __builtin_amdgcn_readfirstlane(first);
      if (want) S.picked[first + (int)__popcll(m & ((1ull << lane) - 1))] = (uint16_t)r;
    }
  };
  BestCut own;   // of the group, in its first lane, or of the lane
  const int gl = t & (kGroup - 1);
  // Where several workgroups share a compute unit (fewer than 1024 threads) its vector ALU is what they wait for, and
  // plain cuts, whose score is short, are scored one lane each once there are more than the groups take at
  // once: 1024 walkers, 32 steps, n = 700 1341 us (by groups alone 1870), n = 442 516 (650), n = 1000 1075 (1363), where
  // few moves are scored, training graph n = 1000, 657 (660).  One workgroup to a compute unit waits for the chain:
  // 64 walkers, n = 442 383 us by groups, 425 with this.
  constexpr bool kByLanes = MODE == 0 && NT < 1024;
  bool by_lanes = false;   // one of the rounds was: any lane may hold the best so far
  auto score_picked = [&](int count) {   // the lane's best to `own`, the group's to `best` in its first lane
    if (kByLanes && count > NT / kGroup) {
      by_lanes = true;
      for (int r = t; r < count; r += NT) {
        const int at = S.picked[r];
        const uint32_t q = S.moves[at], where = S.where[at];
        CutScore sc{};
        Cut c{};
        if (score_cut(lists, C, L, lay, (int)(where >> 16), (int)(where & 0xFFFFu), 0, 0, base_peak, at_peak, true, sc, c) &&
            own.take((uint64_t)(uint32_t)sc.viol << 32 | (uint32_t)sc.peak, (uint64_t)(uint32_t)sc.at << 32 | q))
          cut = c;
      }
    } else {
      for (int r = t / kGroup; r < count; r += NT / kGroup) {
        const int at = S.picked[r];
        const uint32_t q = S.moves[at], where = S.where[at];
        CutScore sc{};
        Cut c{};
        const bool scored = score_cut_by_group<MODE, WIDE>(lists, C, g.parallel != 0, L, lay, (int)(where >> 16), (int)(where & 0xFFFFu),
                                                           base_peak, at_peak, sc, c, gl);
        if (scored && gl == 0) {
          if (own.take((uint64_t)(uint32_t)sc.peak, (uint64_t)(uint32_t)sc.at << 32 | q)) cut = c;
        }
      }
    }
    best = own;
    if (kByLanes && by_lanes) {
#pragma unroll
      for (int off = kGroup / 2; off > 0; off >>= 1)
        best.take((uint64_t)__shfl_xor((unsigned long long)best.score, off), (uint64_t)__shfl_xor((unsigned long long)best.tie, off));
    }
  };
  pick(1, [&](uint32_t bound) { return bucket_of(bound) <= last_bucket; });
  __syncthreads();
  const int first_round = __builtin_amdgcn_readfirstlane(S.counts[1]);
  score_picked(first_round);
  best_of_workgroup<NT, kGroup>(best, L.scratch, t);
  if (first_round < passed) {   // the others, unless their bound lies above what was reached
    const uint64_t reached = best.score;
    pick(3, [&](uint32_t bound) { return bucket_of(bound) > last_bucket && (uint64_t)bound <= reached; });
    __syncthreads();
    const int second_round = __builtin_amdgcn_readfirstlane(S.counts[3]);
    if (second_round > 0) {
      score_picked(second_round);
      best_of_workgroup<NT, kGroup>(best, L.scratch + 4 * NW, t);
    }
  }
  mine_is_best = own.score != ~0ull && own.score == best.score && own.tie == best.tie;
  return true;
}
template <int NT>
__device__ __forceinline__ void clear_sift(const SiftLds& S, int t) {   // before the sieve, a barrier between
  if (t < kBuckets) S.hist[t] = 0;
  if (t < 4) S.counts[t] = t == 2 ? 0x7FFFFFFF : 0;
}

}  // namespace
