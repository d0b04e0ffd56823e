// moc_eval_neighbours: scores every single-field move (start or end of one copy
// by -R..-1, +1..+R positions) of a batch of base candidates.  The move set is
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
// active copies that are not live.  Pass 1 counts the violations of the base
// and marks the copies that take part in one.  Pass 2 runs one lane per (live
// copy, field): it builds the 0/1 terms of f as bit
// masks over the displacements, sums them in bit planes and walks outwards from
// the old position (see build_field, walk_own).  Two kernels: for the best move
// alone (fields that cannot win are left out), and with the table of scores (a
// wave writes the rows of consecutive copies, the inactive ones filled in).
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
  uint32_t* involved;   // bit k: copy k takes part in a violation of Eq. (3) or (5)
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

// A step of moc_search_moves: what the kernel does beyond finding the best move (all null in a plain call).
struct NbSearch {
  int32_t* starts;    // the candidates again, to be edited
  int32_t* ends;
  int32_t* steps;     // per candidate: moves applied
  int32_t* stopped;   // per candidate: its best move does not improve it, and never will
};

// The starts and ends as the kernel reads them.  A step of the descent edits them in the same launch
// (through NbSearch, without the table), so only the instantiations with the table may say that
// nothing else writes them.
template <bool TABLE>
struct Rows { using Ptr = const int32_t* __restrict__; };
template <>
struct Rows<false> { using Ptr = const int32_t*; };

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

template <int kNT, bool ADJ_LDS, int CT, bool WIDE, bool TABLE>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(8, 8))) void neighbours_kernel(GraphView g, int64_t B, typename Rows<TABLE>::Ptr starts,
                                                         typename Rows<TABLE>::Ptr ends,
                                                         const uint8_t* __restrict__ active, int R,
                                                         moc_move_score* __restrict__ out_moves,
                                                         moc_best_move* __restrict__ out_best, NbSearch search,
                                                         NbLayout lay) {
  extern __shared__ uint32_t nb_raw[];
  NbLds L;
  L.profile = reinterpret_cast<int32_t*>(nb_raw);
  L.pmax = L.profile + lay.T_pad + 4;   // pmax[-1] = 0
  L.smax = L.pmax + lay.T_pad;          // smax[T] = 0
  L.packed = reinterpret_cast<uint32_t*>(L.smax + lay.T_pad + 4);
  L.list = reinterpret_cast<uint16_t*>(L.packed + lay.T_pad);
  L.occ1 = reinterpret_cast<uint32_t*>(L.list + lay.T_pad);
  L.occ2 = L.occ1 + lay.bit_words;
  L.involved = L.occ2 + lay.bit_words;
  L.amask = L.involved + lay.mask_words;
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
  int32_t* const counts = L.scratch + 8 * (kNT / kWave);   // [0] base violations, [1] live copies, [2] fewest violations of a move so far, [3] work drawn, [4] active copies that are not live, [5] work drawn from their moves
  const bool pairs = TABLE && (R & 1) == 0 && (reinterpret_cast<uintptr_t>(out_moves) & 15) == 0;   // scores stored two at a time
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
    if constexpr (!TABLE) {
      if (search.stopped && search.stopped[b]) continue;   // the same for the whole workgroup
    }
    // what the staging below derives from the thread index is computed again for every base:
    // kept across bases it would sit in registers that the scoring needs, or be spilled
    int t_ = tid;
    asm volatile("" : "+v"(t_));
    const int lane_ = t_ & (kWave - 1);
    const int wave_ = __builtin_amdgcn_readfirstlane(t_ / kWave);

    const int64_t row = b * T;
    moc_move_score* const row0 = TABLE && out_moves ? out_moves + b * (int64_t)moves_per_cand : nullptr;   // this candidate's table
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
    if (t_ < 6) counts[t_] = t_ == 2 ? 0x7FFFFFFF : 0;
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
        L.involved[k0 >> 5] = (uint32_t)lm;   // the live copies, until pass 1 begins
        L.involved[(k0 >> 5) + 1] = (uint32_t)(lm >> 32);
        atomicAdd(&counts[1], __popcll(lm));
        atomicAdd(&counts[4], __popcll(am & ~lm));
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
    const int n_live = __builtin_amdgcn_readfirstlane(counts[1]), n_ill = __builtin_amdgcn_readfirstlane(counts[4]);
    for (int c = wave_; c < chunks; c += kNW) {
      int both = 0;   // live copies before these 64, and (from bit 16 on) active copies that are not live
      for (int x = lane_; x < c; x += kWave) {
        const int live = __popcll(chunk(L.involved, x));
        both += live + ((__popcll(chunk(L.amask, x)) - live) << 16);
      }
      both = last_lane(scan_sum(both));
      const int before = both & 0xFFFF, before_ill = both >> 16;
      const uint64_t lm = chunk(L.involved, c), ill = chunk(L.amask, c) & ~lm, lower = ((uint64_t)1 << lane_) - 1;
      if ((lm >> lane_) & 1) L.list[before + __popcll(lm & lower)] = (uint16_t)(c * kWave + lane_);
      if ((ill >> lane_) & 1) L.list[n_live + before_ill + __popcll(ill & lower)] = (uint16_t)(c * kWave + lane_);
    }
    block_running_sum<kNT>(L.profile, T, L.scratch, t_);   // Eq. (4) per position
    // For the best move alone the rest looks at the live copies only; the rows of the table are filled
    // by active flags.
    for (int w = t_; w < lay.mask_words; w += kNT) {
      if constexpr (!TABLE) L.amask[w] = L.involved[w];
      L.involved[w] = 0;
    }
    block_max_both_ways<kNT>(L.profile, L.pmax, L.smax, T, L.scratch, t_);

    // ---- pass 1: the violations of the base, each instance once: the copies that are not well formed by
    // their number, per live copy the order pair it opens and its inputs
    if (t_ == 0) viol += n_ill;   // Eq. (2)/(8)
    for (int j = t_; j < n_live; j += kNT) {
      const int k = L.list[j];
      const uint32_t mine = L.packed[k];
      const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic), i = k - v * C;
      const int s = (int)(mine & 0xFFFFu), e = (int)(mine >> 16);
      auto mark = [&](int copy) { atomicOr(&L.involved[copy >> 5], 1u << (copy & 31)); };
      if (bit_at(L.occ2, s)) mark(k);   // Eq. (6): the start is shared
      for (int jj = i + 1; jj < C; ++jj) {   // Eq. (3)
        const uint32_t p = L.packed[v * C + jj];
        if (live_of(p)) {
          if (e > (int)(p & 0xFFFFu)) {
            ++viol;
            mark(k);
            mark(v * C + jj);
          }
          break;
        }
      }
      for (int q = A.in_ptr[v]; q < A.in_ptr[v + 1]; ++q) {   // Eq. (5)
        const int u = A.in_idx[q];
        bool cov = false;
        for (int jj = 0; jj < C; ++jj) cov = cov || covers1(L.packed[u * C + jj], (uint32_t)s);
        if (!cov) {   // the consumer and every copy of the provider could mend it
          ++viol;
          mark(k);
          for (int jj = 0; jj < C; ++jj) mark(u * C + jj);
        }
      }
    }
    int distinct = 0;
    for (int w = t_; w < lay.bit_words; w += kNT) distinct += __popc(L.occ1[w]);
    atomicAdd(&counts[0], viol + nlive - distinct);   // Eq. (6): live copies - distinct starts
    __syncthreads();
    const int base_viol = __builtin_amdgcn_readfirstlane(counts[0]);   // the same in every lane: scalar registers
    const int base_peak = __builtin_amdgcn_readfirstlane(L.pmax[T - 1]);
    // For the best move alone the list is built again, the copies that take part in a violation
    // first: their moves are the ones that can lower the count, and once one has, the others
    // are left out wave by wave (see below).
    int n_first = n_live;   // entries of the list's first part
    if constexpr (!TABLE) {
      int all_first = 0;
      for (int x = lane_; x < chunks; x += kWave) all_first += __popcll(chunk(L.amask, x) & chunk(L.involved, x));
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) all_first += __shfl_xor(all_first, off);
      n_first = __builtin_amdgcn_readfirstlane(all_first);
      for (int c = wave_; c < chunks; c += kNW) {
        int both = 0;
        for (int x = lane_; x < c; x += kWave) {
          const uint64_t am = chunk(L.amask, x), inv = chunk(L.involved, x);
          both += __popcll(am & inv) + (__popcll(am & ~inv) << 16);
        }
        both = last_lane(scan_sum(both));
        const int before_first = both & 0xFFFF, before_rest = both >> 16;
        const uint64_t am = chunk(L.amask, c), inv = chunk(L.involved, c), lower = ((uint64_t)1 << lane_) - 1;
        if ((am & inv) >> lane_ & 1) L.list[before_first + __popcll(am & inv & lower)] = (uint16_t)(c * kWave + lane_);
        if ((am & ~inv) >> lane_ & 1) L.list[n_first + before_rest + __popcll(am & ~inv & lower)] = (uint16_t)(c * kWave + lane_);
      }
      __syncthreads();
    }

    // ---- pass 2: one lane per (live copy, field); the waves draw 64 of these at a time.
    // For the best move alone: start moves first, so that all lanes of a wave run the same
    // field's code.  With the table of scores: both fields of 32 consecutive live copies, and
    // the same wave then fills the rows of the inactive copies between them, so that it
    // writes one contiguous stretch of the table (HBM takes long runs much faster than
    // scattered 128-byte rows).
    Best best{0, 0, -1};
    int published = 0x7FFFFFFF;   // the lane's fewest violations as far as the workgroup has been told
    // (TABLE = false compiles the stores away: fewer registers for the best move alone.  With
    // TABLE the pointer is still tested where it was before the kernel was specialised: the
    // build that knows it to be set orders its waits differently and takes 3.5 ms for the table
    // instead of 3.0.)
    const bool table = TABLE && out_moves != nullptr;
    const int draw = table ? kWave / 2 : kWave;
    const int total = table ? max(n_live, 1) : 2 * n_live;
    for (;;) {
      int u0 = 0;
      if (lane == 0) u0 = atomicAdd(&counts[3], draw);
      u0 = __builtin_amdgcn_readfirstlane(u0);
      if (u0 >= total) break;
      int entry, field;
      if (table) {
        entry = u0 + (lane & 31);
        field = lane >> 5;
      } else {   // both fields of the first part of the list, then both of the rest
        const int u = u0 + lane, part = u >= 2 * n_first ? 1 : 0;
        const int in_part = u - part * 2 * n_first, size = part ? n_live - n_first : n_first;
        field = in_part >= size ? 1 : 0;
        entry = part * n_first + in_part - field * size;
      }
      const bool has_unit = entry < n_live;
      const int k = has_unit ? L.list[entry] : 0;
      const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic), i = k - v * C;
      const int q0 = (2 * k + field) * two_r;
      const int sz = A.size_of(v);
      FieldState<WIDE> st{};
      st.field = -1;
      // For the best move alone, a field none of whose moves can have as few violations as
      // some move already scored (by any wave of the workgroup) is left out.  Before anything
      // is computed for it: a copy that takes part in no violation now (not marked in pass 1,
      // its start not shared) cannot get below the base's count.  After the masks are built:
      // no move has fewer violations than the terms that do not depend on the displacement.
      bool build = has_unit, left_out = false;
      [[maybe_unused]] int least = 0x7FFFFFFF;
      if constexpr (!TABLE) {
        least = *const_cast<volatile int32_t*>(&counts[2]);
        if (build && base_viol > least && !bit_at(L.involved, k) && !bit_at(L.occ2, (int)(L.packed[k] & 0xFFFFu))) {
          build = false;
          left_out = true;
        }
      }
      if (build) build_field<CT, WIDE>(A, C, sz, L, T, R, v, i, field, L.packed[k], base_viol, q0, st);
      bool walk = st.field >= 0;
      if constexpr (!TABLE) walk = walk && st.fixed + min(st.if_live, st.if_dead) <= least;
      if (walk) {
        bool high = false;   // counts above 7 in some lane
#pragma unroll
        for (int p = 3; p < kPlanes; ++p) high = high || Bits<WIDE>::any(st.plane[p]);
        if (high) walk_own<kPlanes, WIDE>(st, L, T, R, out_best != nullptr, pairs, row0, best);
        else walk_own<3, WIDE>(st, L, T, R, out_best != nullptr, pairs, row0, best);
        if constexpr (!TABLE) {
          if (best.move >= 0 && best.viol < published) {
            published = best.viol;
            atomicMin(&counts[2], best.viol);
          }
        }
      }
      if (has_unit && st.field < 0 && !left_out) {   // a node with very many edges (rare): move by move, from scratch
        const int s = starts[row + k], e = ends[row + k];
        const int base_rest = base_viol - node_part(A, C, L.packed, v, i, true, true, s, e);
        for (int d = 0; d < two_r; ++d) {
          const int moved = (field == 0 ? s : e) + (d < R ? d - R : d - R + 1);
          moc_move_score sc{-1, -1};
          if (moved >= 0 && moved < T) {
            score_move(A, C, sz, L, T, v, i, field, s, e, moved, base_rest, base_peak, sc);
            const Best cand{sc.violations, sc.peak, q0 + d};
            if (better(cand, best)) best = cand;
          }
          if (row0) store_score(row0, (uint32_t)(q0 + d), sc);
        }
      }
      if (table) {   // the moves of the inactive copies from this block's first copy to the next block's are not applicable
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
      if (lane == 0) m0 = atomicAdd(&counts[5], kWave);
      m0 = __builtin_amdgcn_readfirstlane(m0);
      if (m0 >= n_ill * four_r) break;
      const int at = m0 + lane;
      if (at < n_ill * four_r) {
        const int j = at / four_r, in_copy = at - j * four_r;
        const int k = L.list[n_live + j], field = in_copy >= two_r ? 1 : 0, d = in_copy - field * two_r;
        const int v = C == 1 ? k : (int)__umulhi((uint32_t)k, c_magic), i = k - v * C;
        const int s = starts[row + k], e = ends[row + k];
        const int moved = (field == 0 ? s : e) + (d < R ? d - R : d - R + 1);
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
        if constexpr (!TABLE) {
          if (search.stopped) {
            // the move is applied if it lowers (violations, max(peak, M), peak); the candidate's rows are
            // read by this workgroup only, and not again in this launch
            const int64_t m1 = max(r.peak, g.budget), m0 = max((int64_t)base_peak, g.budget);
            const bool better_than_now = r.move >= 0 && (r.violations < base_viol || (r.violations == base_viol &&
                                                         (m1 < m0 || (m1 == m0 && r.peak < base_peak))));
            if (better_than_now) {
              const int d = r.move % two_r, field = (r.move / two_r) & 1, k = r.move / four_r;
              (field == 0 ? search.starts : search.ends)[row + k] += d < R ? d - R : d - R + 1;
              search.steps[b] += 1;
            } else {
              search.stopped[b] = 1;
            }
          }
        }
      }
    }
    __syncthreads();
  }
}

using NbKernel = void (*)(GraphView, int64_t, const int32_t*, const int32_t*, const uint8_t*, int, moc_move_score*,
                          moc_best_move*, NbSearch, NbLayout);

// C = 1 and C = 4 have a kernel of their own with 1024 threads only.  Where fewer are taken, C read at
// run time costs less than the threads save (best move, 1024 bases, run time with fewer threads / 1024
// and C fixed: n = 240, C = 1 30 / 51 us, C = 4 54 / 68), but for C = 4 close to T = 2560 (n = 600 109 / 92).
template <int NT, bool ADJ_LDS, bool WIDE, bool TABLE>
NbKernel pick_copies(int C) {
  if constexpr (NT == 1024) {
    if (C == 1) return neighbours_kernel<NT, ADJ_LDS, 1, WIDE, TABLE>;
    if (C == 4) return neighbours_kernel<NT, ADJ_LDS, 4, WIDE, TABLE>;
  }
  switch (C) {
    case 2: return neighbours_kernel<NT, ADJ_LDS, 2, WIDE, TABLE>;
    case 3: return neighbours_kernel<NT, ADJ_LDS, 3, WIDE, TABLE>;
    default: return neighbours_kernel<NT, ADJ_LDS, 0, WIDE, TABLE>;   // C read at run time
  }
}

template <int NT, bool ADJ_LDS>
NbKernel pick_kernel(int C, int R, bool table) {
  if (2 * R > 31) return table ? pick_copies<NT, ADJ_LDS, true, true>(C) : pick_copies<NT, ADJ_LDS, true, false>(C);   // 64-bit displacement masks
  return table ? pick_copies<NT, ADJ_LDS, false, true>(C) : pick_copies<NT, ADJ_LDS, false, false>(C);
}

NbKernel pick_kernel(int nt, bool adj_lds, int C, int R, bool table) {
  switch (nt) {
    case 256: return adj_lds ? pick_kernel<256, true>(C, R, table) : pick_kernel<256, false>(C, R, table);
    case 512: return adj_lds ? pick_kernel<512, true>(C, R, table) : pick_kernel<512, false>(C, R, table);
    default: return adj_lds ? pick_kernel<1024, true>(C, R, table) : pick_kernel<1024, false>(C, R, table);
  }
}

// Threads per base.  A wave scores 64 (copy, field) pairs at a time, and the staging is a chain of
// short passes over T positions: a small base does not feed 16 waves, and several bases on a compute
// unit hide each other's latencies, as long as the batch has several per unit.  Best move alone, R = 8,
// C = 2, microseconds by 256 / 512 / 1024 threads: n = 120, 2048 bases 35 / 52 / 97; n = 442, 1024 bases
// 43 / 45 / 66, 600 bases 42 / 36 / 49, 16 bases 39 / 25 / 26; n = 1000, 1024 bases 91 / 73 / 92, 300
// bases 84 / 48 / 45; n = 1280, 600 bases 104 / 68 / 73; n = 2000, 512 bases 164 / 89 / 71.  With the
// table, 1024 bases: n = 442 90 / 99 / 112, n = 1000 191 / 178 / 208, n = 2000 577 / 376 / 346.
int nb_threads(int T, int64_t B, int num_cu) {
  const int64_t per_cu = (B + num_cu - 1) / num_cu;
  if (T <= 1024 && per_cu >= 4) return 256;
  if (T <= 2560 && per_cu >= 2) return 512;
  return 1024;
}

}  // namespace

namespace {

// One launch over B bases: scores and best moves, or (search) a step of the descent by single-field moves.
int queue_neighbours(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends, const uint8_t* active,
                     int32_t R, moc_move_score* out_moves, moc_best_move* out_best, const NbSearch& search,
                     hipStream_t stream) {
  const int nt = nb_threads(g->view.T, B, g->num_cu);
  const NbLayout lay = nb_layout(g->view.T, g->view.n, g->view.m, g->max_lds, nt);
  const NbKernel kern = pick_kernel(nt, lay.adj_off != 0, g->view.C, R, out_moves != nullptr);
  int per_cu = 0;
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), nt, lay.bytes, false, &per_cu)) return rc;
  const int64_t resident = (int64_t)per_cu * g->num_cu;
  const unsigned grid = (unsigned)(B < resident ? B : resident);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lay.bytes, stream, g->view, B, starts, ends, active, R, out_moves,
                     out_best, search, lay);
  return MOC_OK;
}

// What both calls refuse about the graph: another device, an edge (v,v), a T too large for LDS or for 32-bit offsets.
int check_neighbours(const moc_graph* g, int32_t R) {
  int dev = -1;
  MOC_HIP(hipGetDevice(&dev));
  if (dev != g->device) return MOC_EDEVICE;
  if (g->has_self_loop) return MOC_EINVAL;
  if (nb_layout(g->view.T, g->view.n, g->view.m, g->max_lds, 1024).bytes > g->max_lds) return MOC_EOVERFLOW;
  if ((int64_t)g->view.T * 4 * R * 8 > 0xFFFFFFFFll) return MOC_EOVERFLOW;   // byte offsets in a candidate's table are 32 bits
  return MOC_OK;
}

}  // namespace

extern "C" int moc_eval_neighbours(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends,
                                   const uint8_t* active, int32_t R, moc_move_score* out_moves,
                                   moc_best_move* out_best, void* hip_stream) {
  if (!g || B < 0 || R < 1 || R > 32) return MOC_EINVAL;
  if (!out_moves && !out_best) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (!starts || !ends || !active) return MOC_EINVAL;
  if (((uintptr_t)starts | (uintptr_t)ends) & 3) return MOC_EINVAL;
  if (((uintptr_t)out_moves & 7) || ((uintptr_t)out_best & 7)) return MOC_EINVAL;
  if (const int rc = check_neighbours(g, R)) return rc;
  if (const int rc = queue_neighbours(g, B, starts, ends, active, R, out_moves, out_best, NbSearch{}, static_cast<hipStream_t>(hip_stream)))
    return rc;
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

namespace {

__global__ void start_moves_kernel(int32_t* steps, int32_t* stopped, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  steps[i] = 0;
  stopped[i] = 0;
}

}  // namespace

extern "C" int moc_search_moves(const moc_graph* g, int64_t B, int32_t* starts, int32_t* ends, const uint8_t* active,
                                int32_t R, int32_t max_steps, moc_result* work_results, moc_best_move* work_best,
                                int32_t* out_steps, void* hip_stream) {
  if (!g || B < 0 || max_steps < 0 || R < 1 || R > 32) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (!starts || !ends || !active || !work_results || !work_best || !out_steps) return MOC_EINVAL;
  if ((((uintptr_t)starts | (uintptr_t)ends | (uintptr_t)out_steps) & 3) ||
      (((uintptr_t)work_best | (uintptr_t)work_results) & 7))
    return MOC_EINVAL;
  if (B > 0x7FFFFFFFll) return MOC_EINVAL;
  if (const int rc = check_neighbours(g, R)) return rc;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  // One launch a step: the best-move kernel has the base's own violations and peak, applies the move
  // by itself, and passes over the candidates that have come to their end.  (Before: an evaluation,
  // the best move and an application per step, for every candidate: n = 442, 256 walkers, 16 steps 542 us,
  // now 268; n = 1000, 32 walkers, 8 steps 294 us, now 111.)
  const NbSearch search{starts, ends, out_steps, reinterpret_cast<int32_t*>(work_results)};
  hipLaunchKernelGGL(start_moves_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, stream, out_steps, search.stopped, B);
  for (int step = 0; step < max_steps; ++step)
    if (const int rc = queue_neighbours(g, B, starts, ends, active, R, nullptr, work_best, search, stream)) return rc;
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

