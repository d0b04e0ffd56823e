// What the kernels that score moves of a base candidate share: packed copies, wave scans, and
// the base staged in LDS (copies, memory profile of Eq. (4), maxima over any range of it).
#pragma once

#include "moc_shapes.h"
#include "moc_wave.h"

namespace {

// ------------------------------------------------------------------ packed copies
// s | e << 16; low half 0xFFFF: not live (no position x satisfies 0xFFFF < x).
__device__ __forceinline__ bool live_of(uint32_t p) { return (p & 0xFFFFu) != 0xFFFFu; }
__device__ __forceinline__ bool covers1(uint32_t pu, uint32_t x) { return (pu & 0xFFFFu) < x && (pu >> 16) >= x; }
__device__ __forceinline__ uint32_t pack_copy(bool live, int s, int e) {
  return live ? ((uint32_t)s | ((uint32_t)e << 16)) : MOC_DEAD;
}
__device__ __forceinline__ bool bit_at(const uint32_t* bits, int t) { return (bits[t >> 5] >> (t & 31)) & 1u; }

// LDS written by some lanes of a wave is read by others of the same wave: LDS operations of a
// wave complete in order, so the compiler must keep them in order, and that is all.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------ the base in LDS (MvLayout: moc_shapes.h)
// Adjacency of the graph: in-edges of v are [in_begin(v), in_begin(v + 1)) in the order of in_idx;
// pair(x) = u*C | v*C << 16 of in-edge x; consumers of u are consumer(y), y in [out_begin(u),
// out_begin(u + 1)).  In LDS (16-bit entries) or in global memory.
template <bool LISTS>
struct Lists;
template <>
struct Lists<true> {
  const int32_t* sizes;
  const uint32_t* pairs;
  const uint16_t *in_ptr, *out_ptr, *out_idx;
  __device__ __forceinline__ int in_begin(int v) const { return in_ptr[v]; }
  __device__ __forceinline__ int out_begin(int v) const { return out_ptr[v]; }
  __device__ __forceinline__ int consumer_copy(int y, int) const { return out_idx[y]; }   // w*C
  __device__ __forceinline__ uint32_t pair(int x) const { return pairs[x]; }
  __device__ __forceinline__ int size_of(int v) const { return sizes[v]; }
  template <int NT>
  __device__ __forceinline__ void load(const GraphView& g, uint32_t* at, int t) {
    const int n = g.n, m = g.m, C = g.C;
    int32_t* s = reinterpret_cast<int32_t*>(at);
    uint32_t* p = at + n;
    uint16_t* ip = reinterpret_cast<uint16_t*>(p + m);
    uint16_t* op = ip + n + 1;
    uint16_t* oi = op + n + 1;
    for (int x = t; x < n; x += NT) s[x] = g.size_dur[x].x;
    for (int x = t; x <= n; x += NT) { ip[x] = (uint16_t)g.in_ptr[x]; op[x] = (uint16_t)g.out_ptr[x]; }
    for (int x = t; x < m; x += NT) { p[x] = g.edge_pair_c[x]; oi[x] = (uint16_t)(g.out_idx[x] * C); }
    sizes = s; pairs = p; in_ptr = ip; out_ptr = op; out_idx = oi;
  }
};
template <>
struct Lists<false> {
  GraphView g;
  __device__ __forceinline__ int in_begin(int v) const { return g.in_ptr[v]; }
  __device__ __forceinline__ int out_begin(int v) const { return g.out_ptr[v]; }
  __device__ __forceinline__ int consumer_copy(int y, int C) const { return g.out_idx[y] * C; }
  __device__ __forceinline__ uint32_t pair(int x) const { return g.edge_pair_c[x]; }
  __device__ __forceinline__ int size_of(int v) const { return g.size_dur[v].x; }
  template <int NT>
  __device__ __forceinline__ void load(const GraphView& view, uint32_t*, int) { g = view; }
};

struct BaseLds {
  int32_t *profile, *table, *pre, *suf, *peak_before, *scratch, *marks;   // marks: positions at the peak: how many, the first, the last
  uint32_t *packed, *occ1, *occ2, *peak_bits, *extra;
  __device__ __forceinline__ void carve(uint32_t* raw, const MvLayout& l) {
    profile = reinterpret_cast<int32_t*>(raw);
    table = profile + l.table;
    pre = profile + l.pre;
    suf = profile + l.suf;
    packed = raw + l.packed;
    occ1 = raw + l.occ1;
    occ2 = raw + l.occ2;
    peak_bits = raw + l.peak_bits;
    peak_before = profile + l.peak_before;
    scratch = profile + l.scratch;
    marks = scratch + kScratchWords - 4;
    extra = raw + l.extra;
  }
};

// What one thread saw while staging; summed over the workgroup by the caller.
struct StageSums {
  int viol = 0;   // Eq. (2), (8), (7)
  int live = 0;   // live copies
  int dur = 0;    // Eq. (1)
};

// Stages a candidate: packed copies (an inactive copy is MOC_DEAD, an active one that is not well
// formed MOC_DEAD | 1 << 16), deltas of Eq. (4) in the profile array, start bitmaps.  The first
// loads go out before the arrays are cleared.  Starts with no barrier (the arrays must be free),
// ends with one.
// LOOP: there may be more copies than the threads ask for ahead.
template <int CT, int NT, bool LOOP = true>
__device__ __forceinline__ StageSums stage_copies(const GraphView& g, const BaseLds& L, const MvLayout& lay,
                                                  const int32_t* s_row, const int32_t* e_row, const uint8_t* a_row, int t) {
  constexpr int kAhead = 4;
  const int T = g.T, C = CT ? CT : g.C;
  int as[kAhead], ae[kAhead];
  uint32_t aa[kAhead];
  int2 asd[kAhead];
#pragma unroll
  for (int j = 0; j < kAhead; ++j) {   // lanes past the last copy read it again
    const uint32_t k = (uint32_t)min(j * NT + t, T - 1);
    as[j] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(s_row) + 4u * k);
    ae[j] = *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(e_row) + 4u * k);
    aa[j] = *reinterpret_cast<const uint8_t*>(a_row + k);
    asd[j] = g.size_dur[k / (uint32_t)C];
  }
  for (int x = 4 * t; x < lay.blocks * kBlk; x += 4 * NT) *reinterpret_cast<int4*>(L.profile + x) = make_int4(0, 0, 0, 0);
  for (int w = t; w < lay.bit_words; w += NT) { L.occ1[w] = 0; L.occ2[w] = 0; }
  __syncthreads();
  StageSums sums;
  auto stage = [&](int k, int s, int e, uint32_t flag, int2 sd) {
    const bool act = flag != 0, live = act && (uint32_t)s <= (uint32_t)e && (uint32_t)e < (uint32_t)T;
    L.packed[k] = live ? (uint32_t)s | ((uint32_t)e << 16) : act ? MOC_DEAD | 0x10000u : MOC_DEAD;
    if (k % C == 0 && !act) ++sums.viol;   // Eq. (7)
    if (act) sums.dur += sd.y;
    if (act && !live) ++sums.viol;         // Eq. (2)/(8)
    if (live) {
      ++sums.live;
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
  if constexpr (LOOP)
    for (int k = kAhead * NT + t; k < T; k += NT) stage(k, s_row[k], e_row[k], a_row[k], g.size_dur[k / C]);
  __syncthreads();
  return sums;
}

// The violations of Eq. (3), (5) in the staged base, this thread's share of them.
template <int CT, int NT, typename A>
__device__ __forceinline__ int count_order_and_inputs(const GraphView& g, const A& lists, const uint32_t* __restrict__ packed,
                                                      int t) {
  const int C = CT ? CT : g.C;
  int viol = 0;
  for (int v = t; v < g.n; v += NT) {   // Eq. (3): each live copy against the next live copy of its node
    int end = -1;
    for (int i = 0; i < C; ++i) {
      const uint32_t p = packed[v * C + i];
      if (!live_of(p)) continue;
      viol += end > (int)(p & 0xFFFFu) ? 1 : 0;
      end = (int)(p >> 16);
    }
  }
  for (int x = t; x < g.m; x += NT) {   // Eq. (5): one lane per edge
    const uint32_t pair = lists.pair(x);
    const uint32_t* const pu = packed + (pair & 0xFFFFu);
    const uint32_t* const pv = packed + (pair >> 16);
    for (int i = 0; i < C; ++i) {
      const uint32_t at = pv[i] & 0xFFFFu;
      bool held = at == 0xFFFFu;
      for (int q = 0; q < C; ++q) held = held || covers1(pu[q], at);
      viol += held ? 0 : 1;
    }
  }
  return viol;
}

// profile <- running sums of the profile array (0 behind the last position), and level 0 of the
// table.  A wave takes rows of 256 positions, four per lane.  Ends with a barrier; between(): behind the barrier
// that all threads have met at before (none with one wave).
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <int NT, typename F = Nothing>
__device__ __forceinline__ void scan_profile(const BaseLds& L, const MvLayout& lay, int T, int t, F between = F{}) {
  constexpr int NW = NT / kWave;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int words = lay.blocks * kBlk;
  const int rows = (words + 4 * kWave - 1) / (4 * kWave), per_wave = (rows + NW - 1) / NW;
  const int r0 = min(wave * per_wave, rows), r1 = min(r0 + per_wave, rows);
  int sum = 0;
  for (int r = r0; r < r1; ++r) {
    const int x = (r * kWave + lane) * 4;
    if (x < words) {
      const int4 v = *reinterpret_cast<const int4*>(L.profile + x);
      sum += v.x + v.y + v.z + v.w;
    }
  }
  if constexpr (NW > 1) {
    sum = scan_sum(sum);
    if (lane == kWave - 1) L.scratch[wave] = sum;
    __syncthreads();
  }
  between();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += L.scratch[w];
  for (int r = r0; r < r1; ++r) {
    const int x = (r * kWave + lane) * 4;
    int4 v = make_int4(0, 0, 0, 0);
    if (x < words) v = *reinterpret_cast<const int4*>(L.profile + x);
    v.y += v.x; v.z += v.y; v.w += v.z;
    const int incl = scan_sum(v.w);
    const int base = before + incl - v.w;
    before += last_lane(incl);
    v.x = x < T ? v.x + base : 0;
    v.y = x + 1 < T ? v.y + base : 0;
    v.z = x + 2 < T ? v.z + base : 0;
    v.w = x + 3 < T ? v.w + base : 0;
    int top = max(max(v.x, v.y), max(v.z, v.w));
    top = max(top, __builtin_amdgcn_update_dpp(0, top, 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]: the block's other half
    if (x < words) {
      *reinterpret_cast<int4*>(L.profile + x) = v;
      if ((lane & 1) == 0) L.table[x / kBlk] = top;
    }
  }
  __syncthreads();
}

// The maxima before and from every block, by the last two waves; a barrier before they are read.
template <int NT>
__device__ __forceinline__ void maxima_before_and_from(const BaseLds& L, int blocks, int t) {
  constexpr int NW = NT / kWave;
  const int lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  if (wave == NW - 1) {
    int carry = 0;
    for (int x0 = 0; x0 < blocks; x0 += kWave) {
      const int x = x0 + lane;
      const int incl = max(carry, scan_max(x < blocks ? L.table[x] : 0));
      if (x < blocks) L.pre[x + 1] = incl;
      carry = last_lane(incl);
    }
    if (lane == 0) { L.pre[0] = 0; L.suf[blocks] = 0; }
  }
  if (wave == (NW > 1 ? NW - 2 : 0)) {
    int carry = 0;
    for (int x0 = 0; x0 < blocks; x0 += kWave) {
      const int x = blocks - 1 - (x0 + lane);
      const int incl = max(carry, scan_max(x >= 0 ? L.table[x] : 0));
      if (x >= 0) L.suf[x] = incl;
      carry = last_lane(incl);
    }
  }
}

// The levels of the table above 0, three at a time by all threads (a barrier behind each three), and the
// maxima before and from every block by the last two waves.  Ends with a barrier.  (All levels by one
// wave, one after the other: n = 1000, a step of the descent 1.7 instead of 1.4 us, toggles at n = 2000 111.8
// instead of 109.5.)
template <int NT>
__device__ __forceinline__ void build_maxima(const BaseLds& L, const MvLayout& lay, int t) {
  const int blocks = lay.blocks;
  for (int l = 0; l == 0 || l + 1 < lay.levels; l += 3) {
    const int step = 1 << l;   // blocks an entry of level l stands for
    const int32_t* below = L.table + table_level(l, blocks);
    int32_t* const up1 = L.table + table_level(l + 1, blocks);
    int32_t* const up2 = L.table + table_level(l + 2, blocks);
    int32_t* const up3 = L.table + table_level(l + 3, blocks);
    const int last = blocks - step;   // the level's last entry
    for (int x = t; x + 2 * step <= blocks; x += NT) {
      int v[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) v[d] = below[min(x + d * step, last)];
      const int m2 = max(v[0], v[1]), m4 = max(m2, max(v[2], v[3])), m8 = max(max(m4, max(v[4], v[5])), max(v[6], v[7]));
      up1[x] = m2;
      if (x + 4 * step <= blocks) up2[x] = m4;
      if (x + 8 * step <= blocks) up3[x] = m8;
    }
    if (l == 0) maxima_before_and_from<NT>(L, blocks, t);
    __syncthreads();
  }
}

// profile += change on [lo, hi], level 0 of the table with it.  Ends with a barrier.
// MARK: the positions at which it then reaches `peak` are marked, too (begin_marks before, a barrier between).
struct Range { int lo, hi, change; };
template <int NT, bool MARK, typename R>
__device__ __forceinline__ void add_ranges(const BaseLds& L, const MvLayout& lay, const R* ranges, int count, int peak, int T, int t) {
  for (int x0 = 0; x0 < lay.blocks * kBlk; x0 += 4 * NT) {   // whole waves
    const int x = x0 + 4 * t;
    int4 v = make_int4(0, 0, 0, 0);
    if (x < lay.blocks * kBlk) v = *reinterpret_cast<const int4*>(L.profile + x);
    for (int r = 0; r < count; ++r) {
      const int lo = ranges[r].lo, hi = ranges[r].hi, d = ranges[r].change;
      v.x += lo <= x && x <= hi ? d : 0;
      v.y += lo <= x + 1 && x + 1 <= hi ? d : 0;
      v.z += lo <= x + 2 && x + 2 <= hi ? d : 0;
      v.w += lo <= x + 3 && x + 3 <= hi ? d : 0;
    }
    int top = max(max(v.x, v.y), max(v.z, v.w));
    if (MARK && top >= peak && x < T) {   // few lanes
      const uint32_t hit = ((v.x >= peak ? 1u : 0u) | (v.y >= peak ? 2u : 0u) | (v.z >= peak ? 4u : 0u) | (v.w >= peak ? 8u : 0u)) &
                           (0xFu >> max(x + 4 - T, 0));
      if (hit != 0) {
        atomicOr(&L.peak_bits[x >> 5], hit << (x & 31));
        atomicAdd(&L.marks[0], __popc(hit));
        atomicMin(&L.marks[1], x + __ffs(hit) - 1);
        atomicMax(&L.marks[2], x + 31 - __clz(hit));
      }
    }
    top = max(top, __builtin_amdgcn_update_dpp(0, top, 0xB1, 0xF, 0xF, true));
    if (x < lay.blocks * kBlk) {
      *reinterpret_cast<int4*>(L.profile + x) = v;
      if ((t & 1) == 0) L.table[x / kBlk] = top;
    }
  }
  __syncthreads();
}
__device__ __forceinline__ void clear_marks(const BaseLds& L, int t) {
  if (t == 0) {
    L.marks[0] = 0;
    L.marks[1] = 0x7FFFFFFF;
    L.marks[2] = -1;
  }
}
template <int NT>
__device__ __forceinline__ void begin_marks(const BaseLds& L, const MvLayout& lay, int t) {
  for (int w = t; w < lay.bit_words; w += NT) L.peak_bits[w] = 0;
  clear_marks(L, t);
}

// Maxima of the profile over [lo, hi], 0 <= lo <= hi < T, and over all other positions: whole
// blocks from the tables, the two blocks at the ends position by position.
struct InOut { int in, out; };
// The maximum over `count` >= 1 blocks from `first` on.
__device__ __forceinline__ int blocks_maximum(const BaseLds& L, int blocks, int first, int count) {
  const int level = 31 - __clz(count);
  const int32_t* const row = L.table + ((int)__umul24((uint32_t)level, (uint32_t)blocks + 1u) - (1 << level) + 1);   // table_level
  return max(row[first], row[first + count - (1 << level)]);
}
// v where `on` is all ones or all zeros: v or 0, and the other way round (written out: the compiler makes a
// compare and a select of the second).
__device__ __forceinline__ int where_off(int on, int v) {
  int r;
  asm("v_bfi_b32 %0, %1, 0, %2" : "=v"(r) : "v"(on), "v"(v));
  return r;
}
// Without LEVELS the table has its level 0 only, whose entries between the ends are read one by one: four of them for the
// positions that a move of a live copy changes, more where a copy that was not live takes up its interval, which can
// be the whole domain (n = 4000, C = 2, R = 8, 300 bases, half of the copies ending one position behind it: 163 us, 19500
// with the positions read one by one).
template <bool OUTSIDE, bool LEVELS = true>
__device__ __forceinline__ InOut range_maxima(const BaseLds& L, int blocks, int lo, int hi) {
  const int bl = (int)((uint32_t)lo / kBlk), bh = (int)((uint32_t)hi / kBlk);
  const int4* const fl = reinterpret_cast<const int4*>(L.profile + bl * kBlk);
  const int4* const fh = reinterpret_cast<const int4*>(L.profile + bh * kBlk);
  const int4 l0 = fl[0], l1 = fl[1], h0 = fh[0], h1 = fh[1];
  const int first = bl + 1, count = bh - first;   // whole blocks between
  InOut r{0, 0};
  if constexpr (LEVELS) {
    if (count > 0) r.in = blocks_maximum(L, blocks, first, count);
  } else {
    for (int x = first; x < bh; ++x) r.in = max(r.in, L.table[x]);
  }
  if constexpr (OUTSIDE) r.out = max(L.pre[bl], L.suf[bh + 1]);
  // bit j: position j of the block lies in the range
  uint32_t ml = 0xFFu << (lo & (kBlk - 1)), mh = 0xFFu >> (kBlk - 1 - (hi & (kBlk - 1)));
  if (bl == bh) { ml &= mh; mh = ml; }
  auto take = [&](uint32_t m, int j, int v, int w) {   // positions j and j + 1
    const int on_v = __builtin_amdgcn_sbfe((int)m, j, 1), on_w = __builtin_amdgcn_sbfe((int)m, j + 1, 1);   // all ones or zero
    r.in = max(max(v & on_v, w & on_w), r.in);
    if constexpr (OUTSIDE) r.out = max(max(where_off(on_v, v), where_off(on_w, w)), r.out);
  };
  take(ml, 0, l0.x, l0.y); take(ml, 2, l0.z, l0.w); take(ml, 4, l1.x, l1.y); take(ml, 6, l1.z, l1.w);
  take(mh, 0, h0.x, h0.y); take(mh, 2, h0.z, h0.w); take(mh, 4, h1.x, h1.y); take(mh, 6, h1.z, h1.w);
  return r;
}

// Number of positions in [lo, hi] at which the profile reaches `bound`.  Blocks that stay below it
// are passed over by the levels of the table, the largest run first.
__device__ __forceinline__ int count_reaching(const BaseLds& L, const MvLayout& lay, int lo, int hi, int bound) {
  int count = 0;
  const int last = hi / kBlk;
  for (int b = lo / kBlk; b <= last; ++b) {
    for (int l = lay.levels - 1; l >= 0; --l)
      if (b + (1 << l) <= last + 1 && L.table[table_level(l, lay.blocks) + b] < bound) b += 1 << l;
    if (b > last) break;
    const int4* const at = reinterpret_cast<const int4*>(L.profile + b * kBlk);
    const int4 x = at[0], y = at[1];
    uint32_t m = (x.x >= bound ? 1u : 0u) | (x.y >= bound ? 2u : 0u) | (x.z >= bound ? 4u : 0u) | (x.w >= bound ? 8u : 0u) |
                 (y.x >= bound ? 16u : 0u) | (y.y >= bound ? 32u : 0u) | (y.z >= bound ? 64u : 0u) | (y.w >= bound ? 128u : 0u);
    if (b == lo / kBlk) m &= 0xFFu << (lo & (kBlk - 1));
    if (b == last) m &= 0xFFu >> (kBlk - 1 - (hi & (kBlk - 1)));
    count += __popc(m);
  }
  return count;
}

}  // namespace
