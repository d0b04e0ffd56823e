// The table of moc_eval_neighbours: scores every single-field move (start or end of one copy
// by -R..-1, +1..+R positions) of a batch of base candidates, and picks the best.  The move set is
// this library's (the neighbourhood a local search over the variables of the
// paper's Section 2.1 would scan); each score is, by definition, what
// moc_eval_batch returns for the candidate with that one field changed.
//
// One workgroup per base candidate.  It evaluates the base once and keeps in
// LDS what a move needs: the packed intervals of all copies, the memory profile
// (Eq. (4) left-hand side per position) with its prefix and suffix maxima, and
// two bitmaps of start positions occupied once / more than once (Eq. (6)).
// A move of copy k = (v, i) changes only
//   - whether copy k is well formed                           Eq. (2), (8)
//   - the ordering among the copies of v                      Eq. (3)
//   - the start collision of copy k                           Eq. (6)
//   - the inputs of copy k (in-edges of v)                    Eq. (5), k as consumer
//   - the consumers of v (out-edges of v, all their copies)   Eq. (5), v as provider
//   - the profile on the positions gained or lost             Eq. (4)
// so violations' = violations - f(old copy) + f(new copy) + start-collision delta,
// with f = the first, second, fourth and fifth items counted around node v,
// and peak' = max(prefix max before, suffix max after, shifted profile inside)
// over the changed positions (at most R of them unless the copy was outside
// the domain before the move).
// The live copies are listed while the base is staged, and behind them the
// active copies that are not live.  Pass 1 counts the violations of the base.
// Pass 2 runs one lane per (live copy, field): it builds the 0/1 terms of f as bit
// masks over the displacements, sums them in bit planes and walks outwards from
// the old position (see build_field, walk_own); a wave writes the rows of
// consecutive copies, the inactive ones filled in.  (The best move without the
// table: moc_best_moves.h.)
// The adjacency lists are kept in LDS when that costs no resident workgroup.
#include <algorithm>
#include <type_traits>

#include "moc_moves.h"

namespace {

struct NbLayout {
  int T_pad;      // T rounded up to 4
  int bit_words;  // ceil(T / 32)
  int mask_words; // 2 * ceil(T / 64): the active flags, one bit per copy
  int adj_off;    // word offset of the graph's adjacency lists in LDS, 0 if they stay in global memory
  int bytes;
};

NbLayout nb_layout(int T, int n, int m, int max_lds, int nt) {
  NbLayout l;
  l.T_pad = (T + 3) & ~3;
  l.bit_words = (T + 31) / 32;
  l.mask_words = 2 * ((T + 63) / 64);
  // profile, prefix max, suffix max, packed, the list of copies (16 bits an entry) + bitmaps + scratch
  const int words = 4 * l.T_pad + l.T_pad / 2 + 8 + 2 * l.bit_words + 2 * l.mask_words + 8 * (nt / kWave) + 16;
  l.adj_off = 0;
  const int full = nt == 1024 ? 2 : 4;
  l.bytes = 4 * words;
  // The CSR lists both ways (16-bit entries) and the sizes, which every move reads, if that costs no
  // resident workgroup beyond the fourth (the second of 16 waves).  At T = 4000 it would: with them
  // in LDS and one workgroup of 16 waves per CU the table of scores takes 4.2 ms instead of 3.6; at
  // T = 2000 four workgroups of 512 threads take 73 us (best move, 1024 bases), three with the lists
  // in LDS 90; at T = 884 six workgroups of 256 with the lists 96 us, eight without 101.
  const int with_adj = 4 * (words + n + (2 * (n + 1) + 2 * m + 1) / 2);
  if (m < 0xFFFF && with_adj <= max_lds && std::min(max_lds / with_adj, full) >= std::min(max_lds / l.bytes, full)) {
    l.adj_off = words;
    l.bytes = with_adj;
  }
  return l;
}

// The graph's adjacency, by in-edges and by out-edges (CSR), in LDS or in global memory.
template <bool LDS>
struct Adj {
  using Entry = typename std::conditional<LDS, uint16_t, int32_t>::type;
  const Entry* in_ptr;
  const Entry* in_idx;
  const Entry* out_ptr;
  const Entry* out_idx;
  const int32_t* size;   // m_v, one word per node (LDS) or per two words (the graph's {m_v, w_v} pairs)
  __device__ __forceinline__ int size_of(int v) const { return size[LDS ? v : 2 * v]; }
};

struct NbLds {
  int32_t* profile;
  int32_t* pmax;
  int32_t* smax;
  uint32_t* packed;
  uint16_t* list;   // the live copies, in order, and behind them the active copies that are not live
  uint32_t* occ1;
  uint32_t* occ2;
  uint32_t* lmask;      // bit k: copy k is live
  uint32_t* amask;      // bit k: copy k is active
  int32_t* scratch;   // 8 words per wave + 16
};

// a[x] <- a[0] + ... + a[x].
template <int kNT>
__device__ void block_running_sum(int32_t* a, int T, int32_t* scratch, int tid) {
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int L = (T + kNT - 1) / kNT;
  const int lo = tid * L, hi = min(lo + L, T);
  int acc = 0;
  for (int i = lo; i < hi; ++i) acc += a[i];
  int inc = acc;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int o = __shfl_up(inc, off);
    if (lane >= off) inc += o;
  }
  if (lane == kWave - 1) scratch[wave] = inc;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += scratch[w];
  const int prev = __shfl_up(inc, 1);
  int run = before + (lane == 0 ? 0 : prev);
  for (int i = lo; i < hi; ++i) {
    run += a[i];
    a[i] = run;
  }
  __syncthreads();
}

// dst_up[t] = max(src[0..t]) and dst_down[t] = max(src[t..T-1]) in one pass (src >= 0).
template <int kNT>
__device__ void block_max_both_ways(const int32_t* src, int32_t* dst_up, int32_t* dst_down, int T, int32_t* scratch,
                                    int tid) {
  constexpr int kNW = kNT / kWave;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int L = (T + kNT - 1) / kNT;
  const int lo = tid * L, hi = min(lo + L, T);
  int up = 0, down = 0;
  for (int i = lo; i < hi; ++i) {
    up = max(up, src[i]);
    down = max(down, src[T - 1 - i]);
  }
  int inc_up = up, inc_down = down;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int a = __shfl_up(inc_up, off), b = __shfl_up(inc_down, off);
    if (lane >= off) {
      inc_up = max(inc_up, a);
      inc_down = max(inc_down, b);
    }
  }
  if (lane == kWave - 1) {
    scratch[wave] = inc_up;
    scratch[kNW + wave] = inc_down;
  }
  __syncthreads();
  int run_up = 0, run_down = 0;
  for (int w = 0; w < wave; ++w) {
    run_up = max(run_up, scratch[w]);
    run_down = max(run_down, scratch[kNW + w]);
  }
  const int prev_up = __shfl_up(inc_up, 1), prev_down = __shfl_up(inc_down, 1);
  if (lane != 0) {
    run_up = max(run_up, prev_up);
    run_down = max(run_down, prev_down);
  }
  for (int i = lo; i < hi; ++i) {
    run_up = max(run_up, src[i]);
    dst_up[i] = run_up;
    run_down = max(run_down, src[T - 1 - i]);
    dst_down[T - 1 - i] = run_down;
  }
  __syncthreads();
}

// The part of the violation count that depends on copy i of node v: copy i with the
// given values (all other copies as staged in `packed`).
//   form  : copy i active but not well formed
//   order : Eq. (3) among the live copies of v
//   cons  : in-edges of v not covered at the start of copy i
//   prov  : (out-edge (v,w), live copy of w) pairs not covered by any live copy of v
template <typename A>
__device__ __forceinline__ int node_part(const A& g, int C, const uint32_t* __restrict__ packed, int v, int i,
                                         bool active, bool live, int s, int e) {
  const uint32_t mine = pack_copy(live, s, e);
  int count = (active && !live) ? 1 : 0;
  // Eq. (3): each live copy against the next live copy
  int prev_end = -1;
  bool have_prev = false;
  for (int j = 0; j < C; ++j) {
    const uint32_t p = j == i ? mine : packed[v * C + j];
    if (!live_of(p)) continue;
    if (have_prev && prev_end > (int)(p & 0xFFFFu)) ++count;
    prev_end = (int)(p >> 16);
    have_prev = true;
  }
  // Eq. (5), copy i as consumer
  if (live) {
    for (int q = g.in_ptr[v]; q < g.in_ptr[v + 1]; ++q) {
      const int u = g.in_idx[q];
      bool cov = false;
      for (int j = 0; j < C; ++j) cov = cov || covers1(packed[u * C + j], (uint32_t)s);
      count += cov ? 0 : 1;
    }
  }
  // Eq. (5), node v as provider
  for (int q = g.out_ptr[v]; q < g.out_ptr[v + 1]; ++q) {
    const int w = g.out_idx[q];
    for (int jw = 0; jw < C; ++jw) {
      const uint32_t pw = packed[w * C + jw];
      if (!live_of(pw)) continue;
      const uint32_t x = pw & 0xFFFFu;
      bool cov = false;
      for (int j = 0; j < C; ++j) cov = cov || covers1(j == i ? mine : packed[v * C + j], x);
      count += cov ? 0 : 1;
    }
  }
  return count;
}

// One move of a copy, from scratch: (violations, peak) of the candidate with that one field
// at `moved`.  The general form; the kernel uses it for copies that are ill-formed before
// the move, where the changed positions are a whole interval.
template <typename A>
__device__ __forceinline__ void score_move(const A& g, int C, int sz, const NbLds& L, int T, int v, int i,
                                           int field, int s, int e, int moved, int base_rest, int base_peak,
                                           moc_move_score& sc) {   // base_rest: the base count without f(old copy)
  const int k = v * C + i;
  const int s2 = field == 0 ? moved : s, e2 = field == 0 ? e : moved;
  const bool live_old = live_of(L.packed[k]);
  const bool live_new = (uint32_t)s2 <= (uint32_t)e2 && (uint32_t)e2 < (uint32_t)T;
  int vv = base_rest + node_part(g, C, L.packed, v, i, true, live_new, s2, e2);
  if (live_old && bit_at(L.occ2, s)) --vv;
  if (live_new) vv += (live_old && s2 == s) ? (bit_at(L.occ2, s) ? 1 : 0) : (bit_at(L.occ1, s2) ? 1 : 0);
  // peak: positions lost (sign -1) or gained (sign +1)
  int pk = base_peak;
  if (live_old || live_new) {
    int lo = 0, hi = -1, sign = 0;
    if (live_old && live_new) {
      if (field == 0) { lo = min(s, s2); hi = max(s, s2) - 1; sign = s2 < s ? 1 : -1; }
      else { lo = min(e, e2) + 1; hi = max(e, e2); sign = e2 > e ? 1 : -1; }
    } else if (live_old) { lo = s; hi = e; sign = -1; }
    else { lo = s2; hi = e2; sign = 1; }
    int inside = 0;
    for (int t = lo; t <= hi; ++t) inside = max(inside, L.profile[t] + sign * sz);
    pk = max(inside, max(lo > 0 ? L.pmax[lo - 1] : 0, hi + 1 < T ? L.smax[hi + 1] : 0));
  }
  sc.violations = vv;
  sc.peak = pk;
}

// Sets of moves of one (copy, field) as bit masks.  32 bits serve R <= 15: one bit per
// position first..first+2R around the old one, the old position itself (no move) included.
// 64 bits serve any R this call accepts: one bit per move, d = 0..2R-1 for the displacements
// -R..-1, +1..+R.  below(x, D): the bits under x, clamped to the D bits in use.
template <bool WIDE>
struct Bits;
template <>
struct Bits<false> {
  using M = uint32_t;
  static __device__ __forceinline__ M below(int x, int D) { return (1u << min(max(x, 0), D)) - 1u; }   // D <= 31
  static __device__ __forceinline__ bool any(M m) { return __any(m != 0); }
};
template <>
struct Bits<true> {
  using M = uint64_t;
  static __device__ __forceinline__ M below(int x, int D) {
    const int c = min(x, D);
    return c <= 0 ? 0 : ~(uint64_t)0 >> (64 - c);
  }
  static __device__ __forceinline__ bool any(M m) { return __any(m != 0); }
};

constexpr int kPlanes = 6;           // per-move counters of up to 63 as bit planes; beyond that the slow path
constexpr int kNoCopy = 0x3FFFFFFF;  // start of a copy that does not exist

struct Best {
  int viol, peak, move;   // move < 0: none
};

// Plain stores: a lane writes its row of scores in 16-byte pieces, which the L2 puts together;
// with the non-temporal hint the table takes four times as long.
// `table` is the candidate's table (the same in every lane: a scalar base), `index` the move.
__device__ __forceinline__ void store_score(moc_move_score* table, uint32_t index, const moc_move_score& sc) {
  *reinterpret_cast<moc_move_score*>(reinterpret_cast<char*>(table) + (size_t)(index * 8u)) = sc;
}
__device__ __forceinline__ void store_pair(moc_move_score* table, uint32_t index, const moc_move_score& lo,
                                           const moc_move_score& hi) {   // 16-byte aligned
  *reinterpret_cast<int4*>(reinterpret_cast<char*>(table) + (size_t)(index * 8u)) =
      make_int4(lo.violations, lo.peak, hi.violations, hi.peak);
}

// Order of the best move: (violations, max(peak, budget), peak, move index).  max(peak, budget)
// never decreases with the peak and its ties are broken by the peak, so this is the order
// by (violations, peak, move index).
__device__ __forceinline__ bool better(const Best& a, const Best& b) {
  if (a.move < 0) return false;
  if (b.move < 0) return true;
  if (a.viol != b.viol) return a.viol < b.viol;
  if (a.peak != b.peak) return a.peak < b.peak;
  return a.move < b.move;
}

// What the 2R moves of one field of a live copy add to the violation count, move by move:
// a sum of 0/1 terms, each true on an interval of the moved position.  The terms are built
// as masks over the displacements and summed in bit planes.
template <bool WIDE>
struct FieldState {
  typename Bits<WIDE>::M plane[kPlanes];   // bit d of plane p: bit p of the count of move d
  typename Bits<WIDE>::M live;             // moves that leave the copy well formed
  int fixed, if_live, if_dead;             // violations = fixed + (live ? if_live : if_dead) + count
  int s, e, sz, q0;                        // the copy before the move, its size, index of its first move
  int field;                               // 0: the start moves, 1: the end; -1: nothing to score
};

// The 32-bit masks (R <= 15) have one bit per position first..first+2R, the copy's own
// position (no move) included: the count at that bit is what the copy contributes now, so
// violations of a move = base count - that + count of the move.  The 64-bit masks have one
// bit per move (no room for the extra bit at R = 32); there the copy's present contribution
// is computed edge by edge.  On a counter overflow in any lane the state is marked invalid
// (the caller then scores the moves one by one).
template <int CT, bool WIDE, typename Lists_>
__device__ __forceinline__ void build_field(const Lists_& A, int C, int sz, const NbLds& L, int T, int R, int v, int i,
                                            int field, uint32_t mine, int base_viol, int q0, FieldState<WIDE>& st) {
  using B = Bits<WIDE>;
  using M = typename B::M;
  const int D = WIDE ? 2 * R : 2 * R + 1;
  const int s = (int)(mine & 0xFFFFu), e = (int)(mine >> 16);
  const int base = field == 0 ? s : e, first = base - R;
  // {bits : moved < x}
  auto lt = [&](int x) -> M {
    if constexpr (WIDE) return B::below(x - first - (x > base ? 1 : 0), D);   // moved: first..base-1, base+1..base+R
    else return B::below(x - first, D);                                        // moved: first..base+R
  };
  const M in_dom = lt(T) & ~lt(0);
  const M live = in_dom & (field == 0 ? lt(e + 1) : ~lt(s));   // start <= end after the move
  // Eq. (3): the live neighbours of copy i among the copies of v
  const uint32_t* const row = L.packed + v * C;
  int prev_end = -1, next_start = kNoCopy;
  for (int j = 0; j < C; ++j) {
    const uint32_t p = row[j];
    if (j == i || !live_of(p)) continue;
    if (j < i) prev_end = (int)(p >> 16);
    else if (next_start == kNoCopy) next_start = (int)(p & 0xFFFFu);
  }
  const int start_twice = bit_at(L.occ2, s) ? 1 : 0;
  const int if_dead = 1 + (prev_end > next_start ? 1 : 0);   // Eq. (2)/(8), Eq. (3) across the gap
  int if_live;   // what a move that keeps the copy well formed adds besides the counted terms
  M plane[kPlanes];
#pragma unroll
  for (int p = 0; p < kPlanes; ++p) plane[p] = 0;
  M overflow = 0;
  auto add = [&](M m) {   // most terms are false for every move of every lane
    M carry = m;
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) {
      if (!B::any(carry)) break;
      const M t = plane[p] & carry;
      plane[p] ^= carry;
      carry = t;
    }
    overflow |= carry;
  };
  const int in_lo = A.in_ptr[v], in_hi = A.in_ptr[v + 1];
  if (field == 0) {
    if_live = e > next_start ? 1 : 0;
    add(live & lt(prev_end));   // Eq. (3): the previous copy ends after the new start
    // Eq. (6): the new start is taken (the copy's own start is not a move)
    {
      auto window = [&](int from, int bits) -> M {   // bits of occ1 from position `from` (>= -R) on; positions below 0 read as 0
        const int f0 = max(from, 0), w = min(f0 >> 5, (T - 1) >> 5), w1 = min(w + 1, (T - 1) >> 5);
        const uint64_t two = (uint64_t)L.occ1[w] | ((uint64_t)(w1 > w ? L.occ1[w1] : 0u) << 32);
        return (M)(((two >> (f0 & 31)) << (f0 - from)) & (((uint64_t)1 << bits) - 1));
      };
      if constexpr (WIDE) add(live & (window(first, R) | (window(base + 1, R) << R)));
      else add(live & window(first, D) & ~((M)1 << R));
    }
    // Eq. (5), the copy as consumer: in-edges whose provider does not cover the new start
    for (int q = in_lo; q < in_hi; ++q) {
      const uint32_t* const pu = L.packed + A.in_idx[q] * C;
      M cov = 0;
      for (int j = 0; j < C; ++j) {
        const uint32_t p = pu[j];
        cov |= lt((int)(p >> 16) + 1) & ~lt((int)(p & 0xFFFFu) + 1);   // start < moved <= end; empty for a dead copy
      }
      add(live & ~cov);
    }
  } else {
    add(live & ~lt(next_start + 1));   // Eq. (3): the new end lies after the next copy's start
    int uncovered = 0;                 // Eq. (5), the copy as consumer: the start stays
    for (int q = in_lo; q < in_hi; ++q) {
      const uint32_t* const pu = L.packed + A.in_idx[q] * C;
      bool cov = false;
      for (int j = 0; j < C; ++j) cov = cov || covers1(pu[j], (uint32_t)s);
      uncovered += cov ? 0 : 1;
    }
    if_live = (prev_end > s ? 1 : 0) + start_twice + uncovered;
  }
  // Eq. (5), node v as provider: every live copy of every consumer that no other copy of v covers
  for (int q = A.out_ptr[v], q1 = A.out_ptr[v + 1]; q < q1; ++q) {
    const uint32_t* const pw = L.packed + A.out_idx[q] * C;
    for (int jw = 0; jw < C; ++jw) {
      const int x = (int)(pw[jw] & 0xFFFFu);
      if (x == 0xFFFF) continue;
      bool cov = false;
      for (int j = 0; j < C; ++j) cov = cov || (j != i && covers1(row[j], (uint32_t)x));
      if (cov) continue;
      // the moved copy covers x: start < x <= end
      const M mine_covers = field == 0 ? (x <= e ? live & lt(x) : (M)0) : (s < x ? live & ~lt(x) : (M)0);
      add(in_dom & ~mine_covers);
    }
  }
  // the copy's contribution now, to be replaced by the move's
  int fixed;
  if constexpr (WIDE) {
    int order_others = 0, pe = -1;   // Eq. (3) between other consecutive live copies, on either side of copy i
    for (int j = 0; j < C; ++j) {
      if (j == i) { pe = -1; continue; }
      const uint32_t p = row[j];
      if (!live_of(p)) continue;
      order_others += pe > (int)(p & 0xFFFFu) ? 1 : 0;
      pe = (int)(p >> 16);
    }
    fixed = base_viol - node_part(A, C, L.packed, v, i, true, true, s, e) + order_others - start_twice;
  } else {
    int now = 0;   // the counted terms at the copy's own position
#pragma unroll
    for (int p = 0; p < kPlanes; ++p) now |= (int)((plane[p] >> R) & 1) << p;
    fixed = base_viol - start_twice - now - (if_live - (field == 0 ? 0 : start_twice));
  }
  st.live = live;
  st.fixed = fixed;
  st.if_live = if_live;
  st.if_dead = if_dead;
  st.s = s;
  st.e = e;
  st.sz = sz;
  st.q0 = q0;
  st.field = B::any(overflow) ? -1 : field;
#pragma unroll
  for (int p = 0; p < kPlanes; ++p) st.plane[p] = plane[p];
}

// The lane walks outwards from the old position of its field, one step per displacement on
// either side.  `top` is the maximum of the profile over the positions gained or lost so far
// on a side; a step adds the position that joins the window.  A start moved down or an end
// moved up gains positions, the other two lose them, no further than the other end of the
// interval (the clamp re-reads that end, which changes no maximum).  The peak of a move is
// max(top +- size, prefix maximum before the window, suffix maximum after it); one of the
// two does not change along a side.  NP: bit planes in use.
// The best move of the field is the minimum of violations << 37 | peak << 6 | index of the move
// in the field (violations < 2^26 for any T this call accepts; a move that is not applicable
// has violations -1, the largest key).
template <int NP, bool WIDE>
__device__ __forceinline__ void walk_own(const FieldState<WIDE>& st, const NbLds& L, int T, int R, bool want_best,
                                         bool pairs, moc_move_score* __restrict__ table, Best& best) {
  const int base = st.field == 0 ? st.s : st.e;
  const bool start_moves = st.field == 0;
  // down: a start gains [moved, s-1], an end loses [max(moved+1, s), e]
  const int from_down = base + (start_moves ? 0 : 1), stop_down = start_moves ? 0 : st.s;
  const int size_down = start_moves ? st.sz : -st.sz;
  const int after_down = L.smax[start_moves ? st.s : st.e + 1];
  // up: a start loses [s, min(moved-1, e)], an end gains [e+1, moved]
  const int from_up = base - (start_moves ? 1 : 0), stop_up = start_moves ? st.e : T - 1;
  const int size_up = -size_down;
  const int before_up = L.pmax[(start_moves ? st.s : st.e + 1) - 1];
  const int if_delta = st.if_live - st.if_dead;
  int top_down = 0, top_up = 0;
  uint64_t key = ~(uint64_t)0;
  const int if_dead = st.fixed + st.if_dead;
  auto bit_of = [](typename Bits<WIDE>::M m, int bit) -> int {
    if constexpr (WIDE) return (int)((m >> bit) & 1);
    else return (int)__builtin_amdgcn_ubfe(m, (uint32_t)bit, 1u);
  };
  auto score = [&](int bit, int top, int size, int outside, bool valid, int index) -> moc_move_score {
    int count = if_dead + bit_of(st.live, bit) * if_delta;
#pragma unroll
    for (int p = 0; p < NP; ++p) count += bit_of(st.plane[p], bit) << p;
    moc_move_score sc;
    sc.violations = valid ? count : -1;
    sc.peak = valid ? max(max(top + size, 0), outside) : -1;
    if (want_best) {
      const uint64_t k = ((uint64_t)(uint32_t)sc.violations << 37) | ((uint64_t)(uint32_t)sc.peak << 6) | (uint32_t)index;
      key = k < key ? k : key;
    }
    return sc;
  };
  auto down = [&](int j) -> moc_move_score {
    const int far = max(from_down - j, stop_down);
    top_down = max(top_down, L.profile[far]);
    return score(R - j, top_down, size_down, max(L.pmax[far - 1], after_down), j <= base, R - j);
  };
  auto up = [&](int j) -> moc_move_score {
    const int far = min(from_up + j, stop_up);
    top_up = max(top_up, L.profile[far]);
    return score(WIDE ? R + j - 1 : R + j, top_up, size_up, max(before_up, L.smax[far + 1]), base + j < T, R + j - 1);
  };
  if (pairs) {   // R even, the table 16-byte aligned: two scores per store
    for (int j = 1; j < R; j += 2) {
      const moc_move_score a0 = down(j), b0 = up(j), a1 = down(j + 1), b1 = up(j + 1);
      if (table) {
        store_pair(table, (uint32_t)(st.q0 + R - j - 1), a1, a0);
        store_pair(table, (uint32_t)(st.q0 + R + j - 1), b0, b1);
      }
    }
  } else {
    for (int j = 1; j <= R; ++j) {
      const moc_move_score a0 = down(j), b0 = up(j);
      if (table) {
        store_score(table, (uint32_t)(st.q0 + R - j), a0);
        store_score(table, (uint32_t)(st.q0 + R + j - 1), b0);
      }
    }
  }
  if (want_best && !(key >> 63)) {
    const Best cand{(int)(key >> 37), (int)((key >> 6) & 0x7FFFFFFFu), st.q0 + (int)(key & 63)};
    if (better(cand, best)) best = cand;
  }
}

template <int kNT, bool ADJ_LDS, int CT, bool WIDE>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(8, 8))) void neighbours_kernel(GraphView g, int64_t B, const int32_t* __restrict__ starts,
                                                         const int32_t* __restrict__ ends,
                                                         const uint8_t* __restrict__ active, NbLayout lay, int R,
                                                         moc_move_score* __restrict__ out_moves,
                                                         moc_best_move* __restrict__ out_best) {
  extern __shared__ uint32_t nb_raw[];
  NbLds L;
  L.profile = reinterpret_cast<int32_t*>(nb_raw);
  L.pmax = L.profile + lay.T_pad + 4;   // pmax[-1] = 0
  L.smax = L.pmax + lay.T_pad;          // smax[T] = 0
  L.packed = reinterpret_cast<uint32_t*>(L.smax + lay.T_pad + 4);
  L.list = reinterpret_cast<uint16_t*>(L.packed + lay.T_pad);
  L.occ1 = reinterpret_cast<uint32_t*>(L.list + lay.T_pad);
  L.occ2 = L.occ1 + lay.bit_words;
  L.lmask = L.occ2 + lay.bit_words;
  L.amask = L.lmask + lay.mask_words;
  L.scratch = reinterpret_cast<int32_t*>(L.amask + lay.mask_words);
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int T = g.T, C = CT ? CT : g.C;
  const uint32_t c_magic = 0xFFFFFFFFu / (uint32_t)C + 1u;   // k / C = umulhi(k, c_magic) for C > 1, k < 2^16
  const int two_r = 2 * R, four_r = 4 * R;
  const int moves_per_cand = T * four_r;
  // lane -> move: a wave scores 64 / 4R copies at a time (4R <= 64), or one copy in two pieces
  const int per_wave = four_r <= kWave ? kWave / four_r : 1;
  const int pieces = four_r <= kWave ? 1 : 2;
  const int sub = four_r <= kWave ? lane / four_r : 0;
  const int rem = four_r <= kWave ? lane - sub * four_r : lane;
  int32_t* const counts = L.scratch + 8 * (kNT / kWave);   // [0] base violations, [1] live copies, [2] active copies that are not live, [3] work drawn, [4] work drawn from the moves of the latter
  const bool pairs = (R & 1) == 0 && (reinterpret_cast<uintptr_t>(out_moves) & 15) == 0;   // scores stored two at a time
  constexpr int kNW = kNT / kWave;
  Adj<ADJ_LDS> A;
  if constexpr (ADJ_LDS) {   // the adjacency lists and sizes are read by every move: keep them in LDS
    int32_t* const sizes = reinterpret_cast<int32_t*>(nb_raw) + lay.adj_off;
    uint16_t* const a = reinterpret_cast<uint16_t*>(sizes + g.n);
    for (int x = tid; x <= g.n; x += kNT) { a[x] = (uint16_t)g.in_ptr[x]; a[g.n + 1 + g.m + x] = (uint16_t)g.out_ptr[x]; }
    for (int x = tid; x < g.m; x += kNT) { a[g.n + 1 + x] = (uint16_t)g.in_idx[x]; a[2 * (g.n + 1) + g.m + x] = (uint16_t)g.out_idx[x]; }
    for (int x = tid; x < g.n; x += kNT) sizes[x] = g.size_dur[x].x;
    A = Adj<ADJ_LDS>{a, a + g.n + 1, a + g.n + 1 + g.m, a + 2 * (g.n + 1) + g.m, sizes};
    __syncthreads();
  } else {
    A = Adj<ADJ_LDS>{g.in_ptr, g.in_idx, g.out_ptr, g.out_idx, reinterpret_cast<const int32_t*>(g.size_dur)};
  }

  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    // what the staging below derives from the thread index is computed again for every base:
    // kept across bases it would sit in registers that the scoring needs, or be spilled
    int t_ = tid;
    asm volatile("" : "+v"(t_));
    const int lane_ = t_ & (kWave - 1);
    const int wave_ = __builtin_amdgcn_readfirstlane(t_ / kWave);

    const int64_t row = b * T;
    moc_move_score* const row0 = out_moves + b * (int64_t)moves_per_cand;   // this candidate's table
    // ---- base candidate: stage copies, scatter deltas, mark starts
    // The candidate's first kAhead * kNT copies are asked for before the arrays are cleared, all
    // at once and without conditions (lanes past the last copy read it again): they arrive
    // while the workgroup clears and meets at the barrier, instead of one round of loads
    // after the other, each waited for where it is issued.
    constexpr int kAhead = 4;
    int ahead_s[kAhead], ahead_e[kAhead], ahead_sz[kAhead];
    uint32_t ahead_a[kAhead];
    {
      const char* const s_row = reinterpret_cast<const char*>(starts + row);
      const char* const e_row = reinterpret_cast<const char*>(ends + row);
      const char* const a_row = reinterpret_cast<const char*>(active + row);
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        const uint32_t k = (uint32_t)min(wave_ * kWave + j * kNT + lane_, T - 1);
        ahead_s[j] = *reinterpret_cast<const int32_t*>(s_row + 4u * k);
        ahead_e[j] = *reinterpret_cast<const int32_t*>(e_row + 4u * k);
        ahead_a[j] = *reinterpret_cast<const uint8_t*>(a_row + k);
        ahead_sz[j] = A.size_of(C == 1 ? (int)k : (int)__umulhi(k, c_magic));
      }
    }
    for (int t = t_; t < T; t += kNT) L.profile[t] = 0;
    for (int w = t_; w < 2 * lay.bit_words; w += kNT) L.occ1[w] = 0;   // occ1, occ2
    if (t_ < 5) counts[t_] = 0;
    if (t_ == 0) { L.pmax[-1] = 0; L.smax[T] = 0; }
    __syncthreads();
    // whole waves, 64 consecutive copies each: a ballot gives the active flags of the 64
    int viol = 0, nlive = 0;
    auto stage = [&](int k0, int s, int e, uint32_t flag, int sz) {
      const int k = k0 + lane_;
      bool act = false, live = false;
      if (k < T) {
        act = flag != 0;
        live = act && (uint32_t)s <= (uint32_t)e && (uint32_t)e < (uint32_t)T;
        const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic);
        L.packed[k] = pack_copy(live, s, e);
        if (k == v * C && !act) ++viol;   // Eq. (7)
        if (live) {
          ++nlive;
          atomicAdd(&L.profile[s], sz);
          if (e + 1 < T) atomicSub(&L.profile[e + 1], sz);
          const uint32_t bit = 1u << (s & 31);
          const uint32_t old = atomicOr(&L.occ1[s >> 5], bit);
          if (old & bit) atomicOr(&L.occ2[s >> 5], bit);
        }
      }
      const uint64_t am = __ballot(act), lm = __ballot(live);
      if (lane_ == 0) {
        L.amask[k0 >> 5] = (uint32_t)am;
        L.amask[(k0 >> 5) + 1] = (uint32_t)(am >> 32);
        L.lmask[k0 >> 5] = (uint32_t)lm;
        L.lmask[(k0 >> 5) + 1] = (uint32_t)(lm >> 32);
        atomicAdd(&counts[1], __popcll(lm));
        atomicAdd(&counts[2], __popcll(am & ~lm));
      }
    };
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int k0 = wave_ * kWave + j * kNT;
      if (k0 < T) stage(k0, ahead_s[j], ahead_e[j], ahead_a[j], ahead_sz[j]);
    }
    for (int k0 = wave_ * kWave + kAhead * kNT; k0 < T; k0 += kNT) {
      const int k = min(k0 + lane_, T - 1);
      stage(k0, starts[row + k], ends[row + k], active[row + k], A.size_of(C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic)));
    }
    __syncthreads();
    // the list: the live copies in order, those of 64 copies behind those of the copies before; then,
    // in the same way, the active copies that are not live
    auto chunk = [&](const uint32_t* bits, int c) { return (uint64_t)bits[2 * c] | ((uint64_t)bits[2 * c + 1] << 32); };
    const int chunks = lay.mask_words / 2;
    const int n_live = __builtin_amdgcn_readfirstlane(counts[1]), n_ill = __builtin_amdgcn_readfirstlane(counts[2]);
    for (int c = wave_; c < chunks; c += kNW) {
      int both = 0;   // live copies before these 64, and (from bit 16 on) active copies that are not live
      for (int x = lane_; x < c; x += kWave) {
        const int live = __popcll(chunk(L.lmask, x));
        both += live + ((__popcll(chunk(L.amask, x)) - live) << 16);
      }
      both = last_lane(scan_sum(both));
      const int before = both & 0xFFFF, before_ill = both >> 16;
      const uint64_t lm = chunk(L.lmask, c), ill = chunk(L.amask, c) & ~lm, lower = ((uint64_t)1 << lane_) - 1;
      if ((lm >> lane_) & 1) L.list[before + __popcll(lm & lower)] = (uint16_t)(c * kWave + lane_);
      if ((ill >> lane_) & 1) L.list[n_live + before_ill + __popcll(ill & lower)] = (uint16_t)(c * kWave + lane_);
    }
    block_running_sum<kNT>(L.profile, T, L.scratch, t_);   // Eq. (4) per position
    block_max_both_ways<kNT>(L.profile, L.pmax, L.smax, T, L.scratch, t_);

    // ---- pass 1: the violations of the base, each instance once: the copies that are not well formed by
    // their number, per live copy the order pair it opens and its inputs
    if (t_ == 0) viol += n_ill;   // Eq. (2)/(8)
    for (int j = t_; j < n_live; j += kNT) {
      const int k = L.list[j];
      const uint32_t mine = L.packed[k];
      const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic), i = k - v * C;
      const int s = (int)(mine & 0xFFFFu), e = (int)(mine >> 16);
      for (int jj = i + 1; jj < C; ++jj) {   // Eq. (3)
        const uint32_t p = L.packed[v * C + jj];
        if (live_of(p)) {
          viol += e > (int)(p & 0xFFFFu) ? 1 : 0;
          break;
        }
      }
      for (int q = A.in_ptr[v]; q < A.in_ptr[v + 1]; ++q) {   // Eq. (5)
        const int u = A.in_idx[q];
        bool cov = false;
        for (int jj = 0; jj < C; ++jj) cov = cov || covers1(L.packed[u * C + jj], (uint32_t)s);
        viol += cov ? 0 : 1;
      }
    }
    int distinct = 0;
    for (int w = t_; w < lay.bit_words; w += kNT) distinct += __popc(L.occ1[w]);
    atomicAdd(&counts[0], viol + nlive - distinct);   // Eq. (6): live copies - distinct starts
    __syncthreads();
    const int base_viol = __builtin_amdgcn_readfirstlane(counts[0]);   // the same in every lane: scalar registers
    const int base_peak = __builtin_amdgcn_readfirstlane(L.pmax[T - 1]);
    // ---- pass 2: one lane per (live copy, field); the waves draw both fields of 32 consecutive live copies at
    // a time, and the same wave then fills the rows of the inactive copies between them, so that it
    // writes one contiguous stretch of the table (HBM takes long runs much faster than
    // scattered 128-byte rows).
    Best best{0, 0, -1};
    constexpr int draw = kWave / 2;
    for (;;) {
      int u0 = 0;
      if (lane == 0) u0 = atomicAdd(&counts[3], draw);
      u0 = __builtin_amdgcn_readfirstlane(u0);
      if (u0 >= max(n_live, 1)) break;
      const int entry = u0 + (lane & (draw - 1)), field = lane / draw;
      const bool has_unit = entry < n_live;
      const int k = has_unit ? L.list[entry] : 0;
      const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic), i = k - v * C;
      const int q0 = (2 * k + field) * two_r;
      const int sz = A.size_of(v);
      FieldState<WIDE> st{};
      st.field = -1;
      // (`left_out` is always false.  Without it the compiler spills one register more, inside this loop, where a reload
      // waits behind the table's stores: n = 2000, C = 2, R = 8, 1024 bases 360 instead of 345 us.  Nor is row0 ever null: without
      // the tests of it those take 342, but R = 32, n = 60, 256 bases 48 instead of 46.)
      const bool build = has_unit;
      bool left_out = false;
      if (build) build_field<CT, WIDE>(A, C, sz, L, T, R, v, i, field, L.packed[k], base_viol, q0, st);
      bool walk = st.field >= 0;
      if (walk) {
        bool high = false;   // counts above 7 in some lane
#pragma unroll
        for (int p = 3; p < kPlanes; ++p) high = high || Bits<WIDE>::any(st.plane[p]);
        if (high) walk_own<kPlanes, WIDE>(st, L, T, R, out_best != nullptr, pairs, row0, best);
        else walk_own<3, WIDE>(st, L, T, R, out_best != nullptr, pairs, row0, best);
      }
      if (has_unit && st.field < 0 && !left_out) {   // a node with very many edges (rare): move by move, from scratch
        const int s = starts[row + k], e = ends[row + k];
        const int base_rest = base_viol - node_part(A, C, L.packed, v, i, true, true, s, e);
        for (int d = 0; d < two_r; ++d) {
          const int moved = (int)((uint32_t)(field == 0 ? s : e) + (uint32_t)(d < R ? d - R : d - R + 1));
          moc_move_score sc{-1, -1};
          if (moved >= 0 && moved < T) {
            score_move(A, C, sz, L, T, v, i, field, s, e, moved, base_rest, base_peak, sc);
            const Best cand{sc.violations, sc.peak, q0 + d};
            if (better(cand, best)) best = cand;
          }
          if (row0) store_score(row0, (uint32_t)(q0 + d), sc);
        }
      }
      {   // the moves of the inactive copies from this block's first copy to the next block's are not applicable
        const int k_lo = u0 == 0 ? 0 : (int)L.list[u0];
        const int k_hi = u0 + draw < n_live ? (int)L.list[u0 + draw] : T;
        for (int kk0 = k_lo; kk0 < k_hi; kk0 += per_wave) {
          const int kk = kk0 + sub;
          const bool fill = sub < per_wave && kk < k_hi && !((L.amask[kk >> 5] >> (kk & 31)) & 1u);
          for (int piece = 0; piece < pieces; ++piece) {
            const int in_copy = rem + piece * kWave;
            if (fill && in_copy < four_r) store_score(row0, (uint32_t)(kk * four_r + in_copy), moc_move_score{-1, -1});
          }
        }
      }
    }
    // ---- the moves of the active copies that are not live, one lane per move: most leave the copy as
    // it is, the others make it live (its whole interval joins the profile).  One lane for all 2R
    // moves of a field cost every wave with one such copy 2R times the walk over the node's edges.
    for (;;) {
      int m0 = 0;
      if (lane == 0) m0 = atomicAdd(&counts[4], kWave);
      m0 = __builtin_amdgcn_readfirstlane(m0);
      if (m0 >= n_ill * four_r) break;
      const int at = m0 + lane;
      if (at < n_ill * four_r) {
        const int j = at / four_r, in_copy = at - j * four_r;
        const int k = L.list[n_live + j], field = in_copy >= two_r ? 1 : 0, d = in_copy - field * two_r;
        const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic), i = k - v * C;
        const int s = starts[row + k], e = ends[row + k];
        const int moved = (int)((uint32_t)(field == 0 ? s : e) + (uint32_t)(d < R ? d - R : d - R + 1));
        const int s2 = field == 0 ? moved : s, e2 = field == 0 ? e : moved;
        moc_move_score sc{-1, -1};
        if (moved >= 0 && moved < T) {
          sc = moc_move_score{base_viol, base_peak};
          if ((uint32_t)s2 <= (uint32_t)e2 && (uint32_t)e2 < (uint32_t)T) {
            const int base_rest = base_viol - node_part(A, C, L.packed, v, i, true, false, s, e);
            score_move(A, C, A.size_of(v), L, T, v, i, field, s, e, moved, base_rest, base_peak, sc);
          }
          const Best cand{sc.violations, sc.peak, k * four_r + in_copy};
          if (better(cand, best)) best = cand;
        }
        if (row0) store_score(row0, (uint32_t)(k * four_r + in_copy), sc);
      }
    }
    // ---- best move of the candidate
    if (out_best) {
      // the lane's index, counted here from a full mask: nothing of it is kept in a register
      // across the scoring, and the thread index need not be fetched back behind the table's stores
      const int own = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) << 2;
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) {
        Best o;   // of lane ^ off
        const int from = own ^ (off << 2);
        o.viol = __builtin_amdgcn_ds_bpermute(from, best.viol);
        o.peak = __builtin_amdgcn_ds_bpermute(from, best.peak);
        o.move = __builtin_amdgcn_ds_bpermute(from, best.move);
        if (better(o, best)) best = o;
      }
      if (own == 0) {
        L.scratch[wave_ * 4 + 0] = best.viol;
        L.scratch[wave_ * 4 + 1] = best.peak;
        L.scratch[wave_ * 4 + 2] = best.move;
      }
      __syncthreads();
      if (own == 0 && wave_ == 0) {
        Best all{0, 0, -1};
        for (int w = 0; w < kNW; ++w) {
          const Best o{L.scratch[w * 4], L.scratch[w * 4 + 1], L.scratch[w * 4 + 2]};
          if (better(o, all)) all = o;
        }
        moc_best_move r;
        r.move = all.move;
        r.violations = all.move < 0 ? 0 : all.viol;
        r.peak = all.move < 0 ? 0 : all.peak;
        out_best[b] = r;
      }
    }
    __syncthreads();
  }
}

using NbKernel = void (*)(GraphView, int64_t, const int32_t*, const int32_t*, const uint8_t*, NbLayout, int, moc_move_score*,
                          moc_best_move*);

// C = 1 and C = 4 have a kernel of their own with 1024 threads only.  Where fewer are taken, C read at
// run time costs less than the threads save.
template <int NT, bool ADJ_LDS, bool WIDE>
NbKernel pick_copies(int C) {
  if constexpr (NT == 1024) {
    if (C == 1) return neighbours_kernel<NT, ADJ_LDS, 1, WIDE>;
    if (C == 4) return neighbours_kernel<NT, ADJ_LDS, 4, WIDE>;
  }
  switch (C) {
    case 2: return neighbours_kernel<NT, ADJ_LDS, 2, WIDE>;
    case 3: return neighbours_kernel<NT, ADJ_LDS, 3, WIDE>;
    default: return neighbours_kernel<NT, ADJ_LDS, 0, WIDE>;   // C read at run time
  }
}

NbKernel pick_kernel(int nt, bool adj_lds, int C, int R) {
  const bool wide = 2 * R > 31;   // 64-bit displacement masks
  switch (nt) {
    case 256: return adj_lds ? wide ? pick_copies<256, true, true>(C) : pick_copies<256, true, false>(C)
                             : wide ? pick_copies<256, false, true>(C) : pick_copies<256, false, false>(C);
    case 512: return adj_lds ? wide ? pick_copies<512, true, true>(C) : pick_copies<512, true, false>(C)
                             : wide ? pick_copies<512, false, true>(C) : pick_copies<512, false, false>(C);
    default: return adj_lds ? wide ? pick_copies<1024, true, true>(C) : pick_copies<1024, true, false>(C)
                            : wide ? pick_copies<1024, false, true>(C) : pick_copies<1024, false, false>(C);
  }
}

// Threads per base.  A wave scores 64 (copy, field) pairs at a time, and the staging is a chain of
// short passes over T positions: a small base does not feed 16 waves, and several bases on a compute
// unit hide each other's latencies, as long as the batch has several per unit.  R = 8, C = 2, 1024 bases,
// microseconds by 256 / 512 / 1024 threads: n = 442 90 / 99 / 112, n = 1000 191 / 178 / 208, n = 2000 577 / 376 / 346.  At most
// one base to a compute unit: n = 60, 250 bases 28 / 30 / 32, R = 32, 100 bases 46 / - / 51; n = 128, R = 4, 191 bases 23.5 / 21.1 / 23.9; n = 250, 250 bases 42 / 33 / 32; n =
// 442, 60 bases 60 / 39 / 33.  (C = 4, n = 40, 16 bases 37 with 256, which read C at run time, 33 with 1024.)
int nb_threads(int T, int C, int64_t B, int num_cu) {
  const bool own = C == 2 || C == 3;   // C as a constant with any number of threads
  const int64_t per_cu = (B + num_cu - 1) / num_cu;
  if ((own && T <= 160) || (T <= 1024 && per_cu >= 4)) return 256;
  if ((own && T <= 320) || (T <= 2560 && per_cu >= 2)) return 512;
  return 1024;
}

}  // namespace

// One launch over B bases: the table of scores, and the best moves where they are asked for.
int moc_queue_neighbour_table(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends, const uint8_t* active,
                              int32_t R, moc_move_score* out_moves, moc_best_move* out_best, hipStream_t stream) {
  const int nt = nb_threads(g->view.T, g->view.C, B, g->num_cu);
  const NbLayout lay = nb_layout(g->view.T, g->view.n, g->view.m, g->max_lds, nt);
  const NbKernel kern = pick_kernel(nt, lay.adj_off != 0, g->view.C, R);
  int per_cu = 0;
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), nt, lay.bytes, false, &per_cu)) return rc;
  const int64_t resident = (int64_t)per_cu * g->num_cu;
  const unsigned grid = (unsigned)(B < resident ? B : resident);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lay.bytes, stream, g->view, B, starts, ends, active, lay, R, out_moves,
                     out_best);
  return MOC_OK;
}

