// moc_eval_batch_staged: evaluation in the stage-restricted domain of the paper's Section 2.3
// ("Complexity Reduction by Enforcing an Initial Topological Ordering"), gfx950.
//
// The domain has n(n+1)/2 positions in n stages, stage j holding the j + 1 positions
// j(j+1)/2 .. j(j+1)/2 + j.  A node with place k in the topological order may be computed only
// at slot k of a stage, the first time at slot k of stage k.  A start that is not such a value
// is outside the variable's domain: the copy is treated like one with a position outside the
// domain of Eq. (8) (one violation, used by nothing else, still paid for in Eq. (1)).
// Everything else is Eq. (1)-(8) on those positions.
//
// The domain is far too long for a memory profile in LDS (12.5 M positions at n = 5000), but
// memory can only rise where an interval starts (Section 2.2, memory constraints), and every
// other test compares a start with a start or with an end.  So the kernel renumbers: the
// distinct start positions of the usable copies, in increasing order, become 0, 1, 2, ...
// (at most n*C of them); a start takes the rank of its position, an end the rank of the last
// start position not after it.  Eq. (4) and Eq. (5) keep their outcome under that map; Eq. (2),
// (3), (8) are decided on the positions as given, before the map; for Eq. (6) only copies of
// one node can share a position here (a slot belongs to one node), which a lane sees by itself.
// Ranks without sorting: a usable start is (stage j, node k).  Count the distinct ones per
// stage, prefix-sum the counts over the stages, drop the k of each into its stage's bucket; the
// rank of (j, k) is the bucket's offset plus the number of smaller k in the bucket (buckets
// hold the few nodes recomputed in a stage, and the stage's own node).
//
// One workgroup per candidate at a time, one lane per node, all in LDS.
#include "moc_masks.h"
#include "moc_shapes.h"
#include "moc_wave.h"

namespace {

constexpr int kNT = kStagedThreads;
constexpr int kNW = kNT / kWave;

struct StLayout {
  int cur_off, bucket_off, pj_off, pe_off, delta_off, red_off;   // word offsets
  int chunk;      // delta entries per thread (odd: conflict-free strided reads)
  int bytes;
};

StLayout st_layout(int n, int C) {
  const int T = n * C;
  StLayout l;
  l.chunk = ((T + 1 + kNT - 1) / kNT) | 1;
  l.cur_off = 0;                                   // int32 [n]: per stage count, then end of the stage's bucket
  l.bucket_off = l.cur_off + n;                    // uint16 [T]: node places, stage by stage
  l.pj_off = l.bucket_off + (T + 1) / 2;           // int32 [T]: stage of the copy's start, -1 if not usable; then its record
  l.pe_off = l.pj_off + T;                         // int32 [T]: the copy's end as given
  l.delta_off = l.pe_off + T;                      // int32 [kNT * chunk]
  l.red_off = l.delta_off + kNT * l.chunk;
  l.bytes = 4 * (l.red_off + 8 * kNW + 8);
  return l;
}

// First position of stage j, j < 2^16 (24-bit multiply: full rate).
__device__ __forceinline__ uint32_t stage_start(int j) { return __umul24((uint32_t)j, (uint32_t)j + 1u) >> 1; }

// The stage that holds position p (0 <= p < 2^31): the largest j with j(j+1)/2 <= p.  A
// floating-point estimate, then one exact integer step each way, so that the result does not
// depend on how the square root rounds: the estimate's error stays far below one stage (the
// relative error of the root is a few 2^-24 and the root at most 2^17), so its floor is off by
// one at most.
__device__ __forceinline__ int stage_of(uint32_t p) {
  int j = (int)((__fsqrt_rn(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);
  j = max(j, 0);
  j -= stage_start(j) > p ? 1 : 0;
  j += stage_start(j + 1) <= p ? 1 : 0;
  return j;
}

__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Any C: the copies are read where needed, several passes over them in LDS.
__global__ __launch_bounds__(kNT) void eval_staged_general_kernel(GraphView g, const int32_t* __restrict__ place, int64_t B,
                                                                  const int32_t* __restrict__ starts,
                                                                  const int32_t* __restrict__ ends,
                                                                  const uint8_t* __restrict__ active,
                                                                  moc_result* __restrict__ out, StLayout lay) {
  extern __shared__ uint32_t st_raw[];
  int32_t* const cur = reinterpret_cast<int32_t*>(st_raw + lay.cur_off);
  uint16_t* const bucket = reinterpret_cast<uint16_t*>(st_raw + lay.bucket_off);
  int32_t* const pj = reinterpret_cast<int32_t*>(st_raw + lay.pj_off);
  int32_t* const pe = reinterpret_cast<int32_t*>(st_raw + lay.pe_off);
  int32_t* const delta = reinterpret_cast<int32_t*>(st_raw + lay.delta_off);
  int32_t* const red = reinterpret_cast<int32_t*>(st_raw + lay.red_off);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int n = g.n, C = g.C, T = g.T;
  const uint32_t D = (uint32_t)n * (uint32_t)(n + 1) / 2u;   // positions of the domain

  for (int i = tid; i < kNT * lay.chunk; i += kNT) delta[i] = 0;

  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const int64_t row = b * T;
    for (int j = tid; j < n; j += kNT) cur[j] = 0;
    __syncthreads();

    // ---- per node: Eq. (1), (2), (3), (7), (8) and the domain of the starts; count the distinct
    //      usable starts per stage
    int viol = 0, dur = 0;
    // one copy: i-th of node v (place k, duration w); prev_end = end of the node's latest usable copy so far
    auto copy_step = [&](int v, int k, int w, int i, int s, int e, bool act, int& prev_end) {
      const int c = v * C + i;
      bool live = act && (uint32_t)s <= (uint32_t)e && (uint32_t)e < D;
      int j = -1;
      if (live) {
        j = stage_of((uint32_t)s);
        live = (uint32_t)s - stage_start(j) == (uint32_t)k && (i > 0 || j == k);
      }
      viol += (act && !live) ? 1 : 0;
      if (i == 0) viol += act ? 0 : 1;
      dur += act ? w : 0;
      int code = -1;
      if (live) {
        viol += prev_end > s ? 1 : 0;   // Eq. (3), on the positions as given
        prev_end = e;
        // Eq. (6): a usable start shares its position only with copies of its own node, which
        // sit in the same stage; the first of them stands for the position
        bool first_here = true;
        for (int q = 0; q < i; ++q) first_here = first_here && pj[v * C + q] >> 1 != j;
        if (first_here) atomicAdd(&cur[j], 1);
        else viol += 1;
        code = j << 1 | (first_here ? 1 : 0);
      }
      pj[c] = live ? code : -2;   // -2 >> 1 = -1: no stage
      pe[c] = e;
    };
    for (int v = tid; v < n; v += kNT) {
      const int k = place[v], w = g.size_dur[v].y;
      int prev_end = -1;
      for (int i = 0; i < C; ++i)
        copy_step(v, k, w, i, starts[row + v * C + i], ends[row + v * C + i], active[row + v * C + i] != 0, prev_end);
    }
    __syncthreads();

    // ---- cur[j] <- number of distinct usable starts in stages 0..j (inclusive running sum)
    {
      const int per = (n + kNT - 1) / kNT;
      const int j0 = min(tid * per, n), j1 = min(j0 + per, n);
      int sum = 0;
      for (int j = j0; j < j1; ++j) sum += cur[j];
      int incl = sum;
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
      }
      if (lane == kWave - 1) red[wave] = incl;
      __syncthreads();
      int before = incl - sum;
      for (int w = 0; w < wave; ++w) before += red[w];
      // leave in cur[j] the offset of the stage's bucket: the fill below advances it to the end
      for (int j = j0; j < j1; ++j) {
        const int c = cur[j];
        cur[j] = before;
        before += c;
      }
    }
    __syncthreads();

    // ---- buckets: the place of every node that has a first-at-its-position start in the stage
    for (int v = tid; v < n; v += kNT) {
      const int k = place[v];
      for (int i = 0; i < C; ++i) {
        const int code = pj[v * C + i];
        if (code >= 0 && (code & 1)) bucket[atomicAdd(&cur[code >> 1], 1)] = (uint16_t)k;
      }
    }
    __syncthreads();   // now cur[j] = end of stage j's bucket = start of stage j + 1's

    // ---- renumber, stage the records, scatter Eq. (4)
    for (int v = tid; v < n; v += kNT) {
      const int2 sd = g.size_dur[v];
      const int k = place[v];
      for (int i = 0; i < C; ++i) {
        const int c = v * C + i;
        const int code = pj[c];
        uint32_t rec = MOC_DEAD;
        if (code >= 0) {
          const int j = code >> 1;
          int lo = j ? cur[j - 1] : 0, hi = cur[j];
          int cs = lo;
          for (int x = lo; x < hi; ++x) cs += bucket[x] < k ? 1 : 0;
          // the last start position not after the end: all starts of earlier stages, and those of
          // the end's stage at slots up to the end's
          const uint32_t e = (uint32_t)pe[c];
          const int je = stage_of(e);
          const uint32_t slot_e = e - (uint32_t)je * (uint32_t)(je + 1) / 2u;
          lo = je ? cur[je - 1] : 0;
          hi = cur[je];
          int ce = lo - 1;
          for (int x = lo; x < hi; ++x) ce += bucket[x] <= slot_e ? 1 : 0;
          rec = (uint32_t)cs | (uint32_t)ce << 16;
          atomicAdd(&delta[cs], sd.x);
          atomicSub(&delta[ce + 1], sd.x);
        }
        pj[c] = (int32_t)rec;
      }
    }
    __syncthreads();

    // ---- Eq. (4): peak of the running sum over the renumbered positions
    int S = 0, P = 0;
    {
      int32_t* d = delta + tid * lay.chunk;
      for (int x = 0; x < lay.chunk; ++x) {
        const int y = d[x];
        d[x] = 0;
        S += y;
        P = max(P, S);
      }
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {   // lane l absorbs lanes l+off .. l+2*off-1
        const int S2 = __shfl_down(S, off), P2 = __shfl_down(P, off);
        if (lane + off < kWave) {
          P = max(P, S + P2);
          S += S2;
        }
      }
    }
    // ---- Eq. (5): one lane per edge, every usable copy of the consumer
    for (int x = tid; x < g.m; x += kNT) {
      const uint32_t pair = g.edge_pair_c[x];
      const int kd = (int)(pair >> 16), ub = (int)(pair & 0xFFFFu);
      for (int i = 0; i < C; ++i) {
        const uint32_t pv = (uint32_t)pj[kd + i];
        const uint32_t at = pv & 0xFFFFu;
        bool cov = false;
        for (int q = 0; q < C; ++q) {
          const uint32_t pu = (uint32_t)pj[ub + q];
          cov = cov || ((pu & 0xFFFFu) < at && (pu >> 16) >= at);   // s_u + 1 <= s_v <= e_u; a dead copy has s = 0xFFFF
        }
        viol += (at != 0xFFFFu && !cov) ? 1 : 0;
      }
    }
    viol = wave_sum_i(viol);
    dur = wave_sum_i(dur);
    if (lane == 0) {
      int32_t* r = red + 8 + wave * 4;
      r[0] = S; r[1] = P; r[2] = viol; r[3] = dur;
    }
    __syncthreads();
    if (tid == 0) {
      int S0 = 0, P0 = 0, V = 0, W = 0;
      for (int w = 0; w < kNW; ++w) {
        const int32_t* r = red + 8 + w * 4;
        P0 = max(P0, S0 + r[1]);
        S0 += r[0];
        V += r[2];
        W += r[3];
      }
      moc_result res;
      res.peak = P0;
      res.duration = W;
      res.violations = V;
      res.feasible = (V == 0 && (int64_t)P0 <= g.budget) ? 1 : 0;
      out[b] = res;
    }
    __syncthreads();
  }
}

// C <= 4: the copies of a lane's nodes are held in registers, the workgroup's next candidate is asked
// for as soon as they are used.  U = nodes per lane, at least n / NT (staged_shape).  What the renumbering needs for a
// node's first copy follows from its place k alone: its start can only be slot k of stage k, the
// highest slot of that stage, so that its rank is the last of the stage's; only the copies beyond
// the first, which are few, are put into buckets and searched for.  An end at the last slot of its
// stage (where the first copy of a consumer starts) takes the stage's last rank, any other the
// stage's recomputed nodes up to its slot.  cur[j] holds, in the high bits, first the number of
// distinct recomputed starts of stage j, then the offset of its bucket, then the end of the bucket;
// bit 0 says whether the stage's own node starts there (it comes behind the bucket).
// Bound by the vector ALU (77 %) and by the barriers between the passes.  n = 1000, C = 2, 16384 candidates: 208 us
// with every copy put into a bucket and searched for, correctly rounded square roots and the whole delta array
// scanned; 131 us without these; 103 us with the wave scans and sums by lane shifts instead of the LDS crossbar; 98
// us with predicates as lane masks and violations counted by the scalar unit, the further copies of a lane's nodes
// taken together, and two and a half edges a node (vector instructions per wave and candidate 416 -> 337).
__device__ __forceinline__ int stage_and_slot(uint32_t p, uint32_t* slot) {   // stage_of(p) and the slot in it
  int j = (int)(__builtin_amdgcn_sqrtf(8.0f * (float)p + 1.0f) * 0.5f - 0.5f);   // off by one at most: as in stage_of, with one more ulp (2^-7 at most) in the root
  int at = (int)(p - stage_start(j));
  if (at < 0) {
    at += j;
    --j;
  } else if (at > j) {
    ++j;
    at -= j;
  }
  *slot = (uint32_t)at;
  return j;
}

template <int CT, int NT, int U, int EDGES>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(CT * U <= 4 && U <= 2 && CT <= 3 ? 8 : 4, 8)))
void eval_staged_kernel(GraphView g, const int32_t* __restrict__ place, int64_t B, const int32_t* __restrict__ starts,
                        const int32_t* __restrict__ ends, const uint8_t* __restrict__ active,
                        moc_result* __restrict__ out, SfLayout lay) {
  extern __shared__ uint32_t st_raw[];   // at LDS address 0; the records come first
  constexpr int NW = NT / kWave;
  uint32_t* const rec = st_raw;   // records of the copies; one more node that is never live
  int32_t* const cur = reinterpret_cast<int32_t*>(st_raw + lay.cur_off);
  uint16_t* const bucket = reinterpret_cast<uint16_t*>(st_raw + lay.bucket_off);
  int32_t* const delta = reinterpret_cast<int32_t*>(st_raw + lay.delta_off);
  int32_t* const red = reinterpret_cast<int32_t*>(st_raw + lay.red_off);   // NW words, then four for each wave
  const int tid = threadIdx.x;
  const int n = g.n, T = g.T, m = g.m;
  const uint32_t D = (uint32_t)n * (uint32_t)(n + 1) / 2u;   // positions of the domain

  for (int i = tid; i < NT * lay.chunk; i += NT) delta[i] = 0;
  for (int j = tid; j < n; j += NT) cur[j] = 0;
  if (tid < CT) rec[T + tid] = MOC_DEAD;

  int rs[U][CT], re[U][CT];
  // a node's flags as they lie in memory, in one register, taken apart where they are used:
  // bytes put together in a register as they arrive make each load wait where it is issued
  struct Flags { uint8_t a[CT]; };
  static_assert(sizeof(Flags) <= 4, "the flags of a node fit a register");
  uint32_t ra[U];
  // The candidate's rows are the same for all lanes (scalar registers); a lane adds a 32-bit
  // offset that is formed here from the thread index each time.  Whole addresses per lane, kept
  // across the loop over the candidates, would be spilled, and fetching them back here makes
  // every load of the request wait for the one before.
  struct alignas(4) Ints { int32_t x[CT]; };
  auto request = [&](int64_t cand) {
    const char* const s_row = reinterpret_cast<const char*>(starts + cand * T);
    const char* const e_row = reinterpret_cast<const char*>(ends + cand * T);
    const char* const a_row = reinterpret_cast<const char*>(active + cand * T);
    int t = tid;
    asm volatile("" : "+v"(t));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t off = (uint32_t)min(u * NT + t, n - 1) * CT;   // lanes past the last node re-read it
      const Ints sv = *reinterpret_cast<const Ints*>(s_row + off * 4u);
      const Ints ev = *reinterpret_cast<const Ints*>(e_row + off * 4u);
      const Flags f = *reinterpret_cast<const Flags*>(a_row + off);
#pragma unroll
      for (int i = 0; i < CT; ++i) {
        rs[u][i] = sv.x[i];
        re[u][i] = ev.x[i];
      }
      uint32_t w = 0;
      __builtin_memcpy(&w, &f, sizeof(Flags));
      ra[u] = w;
    }
  };
  if ((int64_t)blockIdx.x < B) request(blockIdx.x);
  // place, m_v, w_v of the lane's nodes and its edges: the same for every candidate
  int rk[U];
  int2 rsd[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int v = min(u * NT + tid, n - 1);
    rk[u] = place[v];
    rsd[u] = g.size_dur[v];
  }
  const uint32_t no_edge = (uint32_t)T | (uint32_t)T << 16;   // beyond the list: the node that is never live
  uint32_t edge[EDGES > 0 ? EDGES : 1];
#pragma unroll
  for (int x = 0; x < EDGES; ++x) {
    const int at = x * NT + tid;
    edge[x] = at < m ? g.edge_pair_c[at] : no_edge;
  }
  __syncthreads();

  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    int t_ = tid;   // what derives from the thread index is formed again for every candidate
    asm volatile("" : "+v"(t_));
    const int lane = t_ & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t_ / kWave);
    // ---- per node: Eq. (1), (2), (3), (7), (8) and the domain of the starts; count the distinct
    //      usable starts per stage.  Predicates are lane masks (moc_masks.h), violations are counted by the
    //      scalar unit.
    int viol = 0;   // of the wave
    int dur = 0, viol_more = 0;
    lanemask in_graph[U], live0[U], more[U][CT];   // lanes with a node; whose first copy is usable; further active copies
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int left = n - (u * NT + wave * kWave);   // the same in all lanes
      in_graph[u] = left >= kWave ? ~(lanemask)0 : left > 0 ? ((lanemask)1 << left) - 1 : 0;
      const lanemask act = byte0_ne_k(ra[u], 0u) & in_graph[u];
      const uint32_t s = (uint32_t)rs[u][0], e = (uint32_t)re[u][0], own = stage_start(rk[u]) + (uint32_t)rk[u];
      live0[u] = act & u_eq(s, own) & u_le(s, e) & u_lt_k(e, D);
      viol += count(in_graph[u] & ~live0[u]);   // Eq. (2), (8) if it is active, Eq. (7) if it is not
      dur += (int)pick(act, (uint32_t)rsd[u].y);
      if (lanes(live0[u])) atomicAdd(&cur[rk[u]], 1);
#pragma unroll
      for (int i = 1; i < CT; ++i) more[u][i] = byte_ne_k(ra[u], i, 0u) & in_graph[u];
    }
    // Further copies are few: those of a lane's first such node and copy are taken together, whatever their place
    // among the lane's (`has`), and the others, which most waves have none of, one by one (`rest`; a start's
    // register then holds the copy's code: stage << 1 | first at its position, -2 if not usable).
    lanemask has = 0, rest = 0, usable = 0, opens = 0;   // opens: it is the first start at its position
    int ps = 0, pe = 0, pk = 0, pat = 0, pj = 0, pw = 0, psz = 0;   // start, end, place, index, stage, duration, size of the one that is taken
    if constexpr (CT > 1) {
      int pend = -1;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 1; i < CT; ++i) {
          const lanemask here = more[u][i] & ~has;
          rest |= more[u][i] & has;
          has |= here;
          if (u == 0 && i == 1) {
            ps = rs[0][1]; pe = re[0][1]; pk = rk[0]; pat = t_ * CT + 1; pw = rsd[0].y; psz = rsd[0].x;
            pend = (int)pick(live0[0], (uint32_t)re[0][0], 0xFFFFFFFFu);
          } else {
            ps = (int)pick(here, (uint32_t)rs[u][i], (uint32_t)ps);
            pe = (int)pick(here, (uint32_t)re[u][i], (uint32_t)pe);
            pat = (int)pick(here, (uint32_t)((u * NT + t_) * CT + i), (uint32_t)pat);
            if (u > 0) {
              pk = (int)pick(here, (uint32_t)rk[u], (uint32_t)pk);
              pw = (int)pick(here, (uint32_t)rsd[u].y, (uint32_t)pw);
              psz = (int)pick(here, (uint32_t)rsd[u].x, (uint32_t)psz);
              pend = (int)pick(here, pick(live0[u], (uint32_t)re[u][0], 0xFFFFFFFFu), (uint32_t)pend);
            }
          }
        }
      if (has != 0) {
        dur += (int)pick(has, (uint32_t)pw);
        const lanemask formed = has & u_le((uint32_t)ps, (uint32_t)pe) & u_lt_k((uint32_t)pe, D);
        uint32_t slot = 0;
        pj = stage_and_slot(pick(formed, (uint32_t)ps), &slot);
        usable = formed & u_eq(slot, (uint32_t)pk);
        // Eq. (6): a usable start shares its position only with copies of its own node, which sit in the same stage;
        // the first of them stands for the position.  Eq. (3) on the positions as given.
        opens = usable & ~(~u_eq((uint32_t)pend, 0xFFFFFFFFu) & u_eq((uint32_t)pj, (uint32_t)pk));
        viol += count(has & ~usable) + count(usable & ~opens) + count(usable & i_gt((uint32_t)pend, (uint32_t)ps));
        if (lanes(opens)) atomicAdd(&cur[pj], 2);
      }
      if (rest != 0) {
        lanemask before = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          int end = (int)pick(live0[u], (uint32_t)re[u][0], 0xFFFFFFFFu);   // of the node's latest usable copy so far
          int code[CT];
          code[0] = (int)pick(live0[u], (uint32_t)(rk[u] << 1), 0xFFFFFFFEu);
#pragma unroll
          for (int i = 1; i < CT; ++i) {
            const lanemask taken = more[u][i] & ~before;   // done above
            const lanemask mine = more[u][i] & before;
            before |= more[u][i];
            const int s = rs[u][i], e = re[u][i];
            code[i] = (int)pick(taken & usable, (uint32_t)(pj << 1), 0xFFFFFFFEu);
            if (lanes(mine)) {
              dur += rsd[u].y;
              const bool formed = (uint32_t)s <= (uint32_t)e && (uint32_t)e < D;
              uint32_t slot = 0;
              const int j = stage_and_slot(formed ? (uint32_t)s : 0u, &slot);
              if (formed && slot == (uint32_t)rk[u]) {
                bool first_here = true;
#pragma unroll
                for (int q = 0; q < i; ++q) first_here = first_here && code[q] >> 1 != j;
                if (first_here) atomicAdd(&cur[j], 2);
                code[i] = j << 1 | (first_here ? 1 : 0);
                viol_more += (first_here ? 0 : 1) + (end > s ? 1 : 0);
              } else {
                viol_more += 1;   // Eq. (2), (8)
              }
            }
            rs[u][i] = code[i];
            if (code[i] >= 0) end = e;
          }
        }
        viol += last_lane(scan_sum(viol_more));
      }
    }
    __syncthreads();

    // ---- cur[j] <- offset of the stage's bucket, by a running sum of the starts in the stages before
    int total;   // distinct usable starts
    {
      const int j0 = t_ * U;
      int c[U], sum = 0;
#pragma unroll
      for (int d = 0; d < U; ++d) {
        c[d] = j0 + d < n ? cur[j0 + d] : 0;
        sum += (c[d] >> 1) + (c[d] & 1);
      }
      const int incl = scan_sum(sum);
      if (lane == kWave - 1) red[wave] = incl;
      __syncthreads();
      const int upto = scan_sum_first<NW>(lane < NW ? red[lane] : 0);   // lane w: the waves up to w
      total = __builtin_amdgcn_readlane(upto, NW - 1);
      int before = incl - sum + (wave == 0 ? 0 : __builtin_amdgcn_readlane(upto, wave - 1));
#pragma unroll
      for (int d = 0; d < U; ++d) {
        if (j0 + d < n) cur[j0 + d] = before << 1 | (c[d] & 1);
        before += (c[d] >> 1) + (c[d] & 1);
      }
    }
    __syncthreads();

    // ---- buckets: the place of every node that is computed again in the stage
    if constexpr (CT > 1) {
      if (lanes(opens)) bucket[atomicAdd(&cur[pj], 2) >> 1] = (uint16_t)pk;
      if (rest != 0) {
        lanemask before = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 1; i < CT; ++i) {
            const lanemask mine = more[u][i] & before;
            before |= more[u][i];
            const int code = rs[u][i];
            if (lanes(mine))
              if (code >= 0 && (code & 1)) bucket[atomicAdd(&cur[code >> 1], 2) >> 1] = (uint16_t)rk[u];
          }
      }
      __syncthreads();
    }

    // ---- renumber, stage the records, scatter Eq. (4)
    // recomputed nodes of stage j with a place below `bound`, on top of the rank of the stage's first start
    auto rank_in_stage = [&](int j, uint32_t bound) -> int {
      const int before = j ? cur[j - 1] : 0, hi = cur[j] >> 1;
      const int lo = (before >> 1) + (before & 1);
      int r = lo;
      for (int x = lo; x < hi; ++x) r += bucket[x] < bound ? 1 : 0;
      return r;
    };
    auto rank_of_end = [&](uint32_t e) -> int {   // of the last start not after position e
      uint32_t slot;
      const int j = stage_and_slot(e, &slot);
      if (slot == (uint32_t)j) {
        const int c = cur[j];
        return (c >> 1) + (c & 1) - 1;
      }
      return rank_in_stage(j, slot + 1) - 1;
    };
    auto settle = [&](int cs, uint32_t e, int size) -> uint32_t {
      const int ce = rank_of_end(e);
      atomicAdd(&delta[cs], size);
      atomicSub(&delta[ce + 1], size);
      return (uint32_t)cs | (uint32_t)ce << 16;
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (in_graph[u] == 0) continue;
      const int v = u * NT + t_;
      uint32_t r = MOC_DEAD;
      if (lanes(live0[u])) r = settle(cur[rk[u]] >> 1, (uint32_t)re[u][0], rsd[u].x);
      if (lanes(in_graph[u])) {
        rec[v * CT] = r;
#pragma unroll
        for (int i = 1; i < CT; ++i) rec[v * CT + i] = MOC_DEAD;
      }
    }
    if constexpr (CT > 1) {   // (LDS operations of a wave complete in order: behind the words above)
      if (lanes(usable)) rec[pat] = settle(rank_in_stage(pj, (uint32_t)pk), (uint32_t)pe, psz);
      if (rest != 0) {
        lanemask before = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 1; i < CT; ++i) {
            const lanemask mine = more[u][i] & before;
            before |= more[u][i];
            if (lanes(mine))
              if (rs[u][i] >= 0) rec[(u * NT + t_) * CT + i] = settle(rank_in_stage(rs[u][i] >> 1, (uint32_t)rk[u]), (uint32_t)re[u][i], rsd[u].x);
          }
      }
    }
    if (b + gridDim.x < B) request(b + gridDim.x);   // the rest of this turn works from LDS
    __syncthreads();

    // ---- Eq. (4): peak of the running sum over the renumbered positions (the releases behind the
    // last of them change no maximum but are cleared)
    int S = 0, P = 0;
    {
      const int chunk = ((total + 1 + NT - 1) / NT) | 1;   // <= lay.chunk
      int own = t_;
      asm volatile("" : "+v"(own));
      int32_t* d = delta + own * chunk;
      for (int x = 0; x < chunk; ++x) {
        const int y = d[x];
        d[x] = 0;
        S += y;
        P = max(P, S);
      }
      combine_segments(S, P);
    }
    for (int j = t_; j < n; j += NT) cur[j] = 0;   // for the next candidate
    // ---- Eq. (5): one lane per edge, every usable copy of the consumer
    auto check = [&](uint32_t pair) {
      Record<CT> pu, pv;
      const uint32_t ua = (pair & 0xFFFFu) << 2, va = pair >> 16 << 2;   // LDS addresses
      if constexpr (CT == 2) {
        const uint2 a = lds_read2(ua), c = lds_read2(va);
        pu.w[0] = a.x; pu.w[1] = a.y; pv.w[0] = c.x; pv.w[1] = c.y;
      } else {
#pragma unroll
        for (int q = 0; q < CT; ++q) {
          pu.w[q] = lds_read(ua + 4 * q);
          pv.w[q] = lds_read(va + 4 * q);
        }
      }
#pragma unroll
      for (int i = 0; i < CT; ++i) viol += count(live_uncovered_lanes<CT>(pu, pv.w[i]));
    };
    if constexpr (EDGES > 0) {
#pragma unroll
      for (int x = 0; x < EDGES; ++x) check(edge[x]);
    } else {
      for (int x0 = 0; x0 < m; x0 += NT) {   // every lane the same number of rounds
        const uint32_t pair = g.edge_pair_c[min(x0 + t_, m - 1)];
        check(x0 + t_ < m ? pair : no_edge);
      }
    }
    dur = scan_sum(dur);
    if (lane == kWave - 1)   // the lane that holds the wave's totals
      *reinterpret_cast<int4*>(red + 16 + wave * 4) = make_int4(S, P, viol, dur);
    __syncthreads();
    // (no barrier behind this: the words read here are written again behind several)
    if (wave == 0) {
      int4 r = *reinterpret_cast<const int4*>(red + 16 + min(lane, NW - 1) * 4);
      combine_first<NW>(r.x, r.y);
      const int V = scan_sum_first<NW>(r.z), W = scan_sum_first<NW>(r.w);
      if (lane == NW - 1) {
        moc_result res;
        res.peak = r.y;
        res.duration = W;
        res.violations = V;
        res.feasible = (V == 0 && (int64_t)r.y <= g.budget) ? 1 : 0;
        out[b] = res;
      }
    }
  }
}

using StagedKernel = void (*)(GraphView, const int32_t*, int64_t, const int32_t*, const int32_t*, const uint8_t*, moc_result*, SfLayout);

// The edges of a lane stay in registers where there are at most three to a node (of two and a half a sixth less is padding).
template <int CT, int NT, int U>
StagedKernel pick_edges(int m) {
  const int per_lane = (m + NT - 1) / NT;
  if (per_lane <= 5 * U / 2) return eval_staged_kernel<CT, NT, U, 5 * U / 2>;
  if (per_lane <= 3 * U) return eval_staged_kernel<CT, NT, U, 3 * U>;
  return eval_staged_kernel<CT, NT, U, 0>;
}
template <int NT, int U>
StagedKernel pick_copies(int C, int m) {
  switch (C) {
    case 1: return pick_edges<1, NT, U>(m);
    case 2: return pick_edges<2, NT, U>(m);
    case 3: if constexpr (U <= 2) return pick_edges<3, NT, U>(m); else return nullptr;
    case 4: if constexpr (U <= 2) return pick_edges<4, NT, U>(m); else return nullptr;
    default: return nullptr;
  }
}
template <int NT>
StagedKernel pick_nodes(int nodes, int C, int m) {
  return nodes == 1 ? pick_copies<NT, 1>(C, m) : pick_copies<NT, 2>(C, m);
}
StagedKernel pick_kernel(const StagedShape& shape, int C, int m) {
  switch (shape.nt) {
    case 64: return pick_nodes<64>(shape.nodes, C, m);
    case 128: return pick_nodes<128>(shape.nodes, C, m);
    case 256: return pick_nodes<256>(shape.nodes, C, m);
    case 512: return pick_nodes<512>(shape.nodes, C, m);
    case 1024: return shape.nodes == 4 ? pick_copies<1024, 4>(C, m) : pick_copies<1024, 2>(C, m);
    default: return nullptr;
  }
}

}  // namespace

extern "C" int moc_eval_batch_staged(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends,
                                     const uint8_t* active, moc_result* out, void* hip_stream) {
  if (!g || B < 0) return MOC_EINVAL;
  if (!g->place) return MOC_EINVAL;   // moc_graph_set_order has not been called
  if (B == 0) return MOC_OK;
  if (!starts || !ends || !active || !out) return MOC_EINVAL;
  if ((((uintptr_t)starts | (uintptr_t)ends) & 3) || ((uintptr_t)out & 7)) return MOC_EINVAL;
  int dev = -1;
  MOC_HIP(hipGetDevice(&dev));
  if (dev != g->device) return MOC_EDEVICE;
  const StLayout lay = st_layout(g->view.n, g->view.C);
  if (lay.bytes > g->max_lds || g->view.T >= 0xFFFF) return MOC_EOVERFLOW;
  const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const StagedShape shape = staged_shape(g->view.n, g->view.C, B, g->num_cu);
  const bool in_registers = shape.nodes > 0;
  const int nt = shape.nt;
  const StagedKernel kern = in_registers ? pick_kernel(shape, g->view.C, g->view.m) : nullptr;
  if (in_registers && !kern) return MOC_EINVAL;
  const SfLayout sf = sf_layout(g->view.n, g->view.C, nt);
  const int bytes = in_registers ? sf.bytes : lay.bytes;
  const void* const entry = in_registers ? reinterpret_cast<const void*>(kern) : reinterpret_cast<const void*>(eval_staged_general_kernel);
  int per_cu = 0;
  if (const int rc = moc_kernel_occupancy(g, entry, nt, bytes, in_registers, &per_cu)) return rc;
  const int64_t resident = (int64_t)per_cu * g->num_cu;
  const unsigned grid = (unsigned)(B < resident ? B : resident);
  if (in_registers)
    hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), bytes, stream, g->view, g->place, B, starts, ends, active, out, sf);
  else
    hipLaunchKernelGGL(eval_staged_general_kernel, dim3(grid), dim3(nt), bytes, stream, g->view, g->place, B, starts, ends, active, out, lay);
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}
