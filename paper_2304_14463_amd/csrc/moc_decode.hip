// moc_decode_batch: from candidate assignments back to the rematerialisation sequences they
// stand for, with each sequence's own cost (gfx950).
//
// Section 2 of the paper (arXiv 2304.14463): the start of an active interval is the event at
// which its node is computed, so the active copies read in order of their starts are the
// sequence.  Section 1 (problem statement): a sequence is valid when every node occurs and the
// outputs of all predecessors of a node are in memory when it is computed; it costs the summed
// duration and the peak footprint.  The footprint taken here is the sequence's own: a use is
// served by the most recent earlier computation of the producer, an output is held from its
// step through the last step it serves.
//
// One workgroup per candidate, everything in LDS.  Starts are distinct (otherwise the
// candidate is not decodable), so sorting is a scatter by start followed by a prefix count of
// the occupied positions; the footprint is computed over positions rather than steps -- an
// empty position holds a subset of what the next step holds -- by the same difference array
// and running sum as Eq. (4).
#include <algorithm>

#include "moc_masks.h"
#include "moc_shapes.h"
#include "moc_wave.h"

namespace {

constexpr int kNT = kDecodeThreads;
constexpr int kNW = kNT / kWave;
constexpr uint32_t kNoStart = 0xFFFFu;

// Both scans below walk the array in rows of 64 consecutive positions, one lane per position
// (no bank conflicts); wave w owns the rows [w * rows_per_wave, (w + 1) * rows_per_wave).

// a[x] in {0, 1}: a[x] <- number of ones before x, for x in [0, T); returns the number of ones.
// Every thread of the workgroup calls it; ends with a barrier.
__device__ int block_rank_of_ones(int32_t* a, int T, int32_t* scratch, int tid) {
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int rows = (T + kWave - 1) / kWave, rows_per_wave = (rows + kNW - 1) / kNW;
  const int r0 = min(wave * rows_per_wave, rows), r1 = min(r0 + rows_per_wave, rows);
  int carry = 0;
  for (int r = r0; r < r1; ++r) {
    const int x = r * kWave + lane;
    const bool one = x < T && a[x] != 0;
    const uint64_t ones = __ballot(one);
    if (x < T) a[x] = carry + __popcll(ones & ((1ull << lane) - 1));
    carry += __popcll(ones);
  }
  if (lane == 0) scratch[wave] = carry;
  __syncthreads();
  int before = 0, total = 0;
  for (int w = 0; w < kNW; ++w) {
    const int t = scratch[w];
    if (w < wave) before += t;
    total += t;
  }
  if (before)
    for (int r = r0; r < r1; ++r) {
      const int x = r * kWave + lane;
      if (x < T) a[x] += before;
    }
  __syncthreads();
  return total;
}

// max over x in [0, T) of a[0] + ... + a[x] (at least 0).  Ends with a barrier.
__device__ int block_peak_of_running_sum(const int32_t* a, int T, int32_t* scratch, int tid) {
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int rows = (T + kWave - 1) / kWave, rows_per_wave = (rows + kNW - 1) / kNW;
  const int r0 = min(wave * rows_per_wave, rows), r1 = min(r0 + rows_per_wave, rows);
  int carry = 0, top = INT32_MIN;   // sum and highest running sum of this wave's rows, from the wave's first position
  for (int r = r0; r < r1; ++r) {
    const int x = r * kWave + lane;
    const int inc = scan_sum(x < T ? a[x] : 0);
    top = max(top, carry + inc);
    carry += __builtin_amdgcn_readlane(inc, kWave - 1);
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) top = max(top, __shfl_xor(top, off));
  if (lane == 0) {
    scratch[wave] = carry;
    scratch[kNW + wave] = top;
  }
  __syncthreads();
  int best = 0, before = 0;
  for (int w = 0; w < kNW; ++w) {
    const int t = scratch[kNW + w];
    if (t != INT32_MIN) best = max(best, before + t);
    before += scratch[w];
  }
  __syncthreads();
  return best;
}

// Loops over copies, nodes and edges run the same number of rounds in every lane, kUnroll
// items per lane and round, and read what they need from global memory at the top of a round:
// the loads of a round are in flight together instead of one behind the other.
constexpr int kUnroll = 4;

__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(8, 8)))
void decode_kernel(GraphView G, int64_t B, const int32_t* __restrict__ starts, const uint8_t* __restrict__ active,
                   moc_decode_result* __restrict__ out, int32_t* __restrict__ out_seq, DcLayout lay) {
  extern __shared__ int32_t lds[];
  int32_t* a = lds;                 // occupancy, then step number, then memory differences, per position
  int32_t* b = a + lay.T_pad;       // the sequence, then the last position each computation serves
  uint16_t* st = reinterpret_cast<uint16_t*>(b + lay.T_pad);   // start of each copy, kNoStart if inactive
  int32_t* scratch = reinterpret_cast<int32_t*>(st + lay.T_pad);
  int32_t* flags = scratch + 2 * kNW;   // [0] not decodable, [1] not a valid sequence, [2] duration
  const int tid = threadIdx.x, T = G.T, n = G.n, C = G.C, m = G.m;

  for (int64_t cand = blockIdx.x; cand < B; cand += gridDim.x) {
    const int32_t* s_row = starts + cand * T;
    const uint8_t* a_row = active + cand * T;
    int32_t* seq_row = out_seq ? out_seq + cand * T : nullptr;

    for (int x = tid; x <= T; x += kNT) a[x] = 0;
    if (tid < 4) flags[tid] = 0;
    __syncthreads();

    // scatter by start: a[x] = 1 where a computation happens
    for (int round = 0; round < T; round += kUnroll * kNT) {
      const int base = round + tid;
      // loads without conditions (lanes past the last copy read it again), a register per flag:
      // under a condition, or packed into one register, each load waits for the one before
      uint32_t on[kUnroll];
      int32_t s[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int k = min(base + u * kNT, T - 1);
        on[u] = a_row[k];
        s[u] = s_row[k];
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int k = base + u * kNT;
        if (k >= T) continue;
        uint32_t sk = kNoStart;
        if (on[u]) {
          if (s[u] < 0 || s[u] >= T) {
            flags[0] = 1;                       // Eq. (8)
          } else {
            sk = (uint32_t)s[u];
            if (atomicAdd(&a[s[u]], 1) != 0) flags[0] = 1;   // Eq. (6)
          }
        }
        st[k] = (uint16_t)sk;
      }
    }
    __syncthreads();
    if (flags[0]) {
      if (seq_row)
        for (int x = tid; x < T; x += kNT) seq_row[x] = -1;
      if (tid == 0) out[cand] = moc_decode_result{-1, 0, 0, 0};
      __syncthreads();
      continue;
    }

    // step number of each occupied position
    const int length = block_rank_of_ones(a, T, scratch, tid);

    if (seq_row) {
      for (int v = tid; v < n; v += kNT)
        for (int i = 0; i < C; ++i) {
          const uint32_t p = st[v * C + i];
          if (p != kNoStart) b[a[p]] = v;
        }
      for (int x = length + tid; x < T; x += kNT) b[x] = -1;
      __syncthreads();
      for (int x = tid; x < T; x += kNT) seq_row[x] = b[x];
      __syncthreads();
    }

    // every computation serves at least its own step; the difference array starts at zero
    for (int x = tid; x <= T; x += kNT) a[x] = 0;
    for (int k = tid; k < T; k += kNT) {
      const uint32_t p = st[k];
      if (p != kNoStart) b[p] = (int)p;
    }
    __syncthreads();

    // one lane per edge (u, v): each computation of v is served by the latest computation of u before it
    for (int round = 0; round < m; round += kUnroll * kNT) {
      const int base = round + tid;
      uint32_t pair[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) pair[u] = base + u * kNT < m ? G.edge_pair_c[base + u * kNT] : 0u;
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if (base + u * kNT >= m) continue;
        const int uC = (int)(pair[u] & 0xFFFFu), vC = (int)(pair[u] >> 16);
        for (int i = 0; i < C; ++i) {
          const uint32_t p = st[vC + i];
          if (p == kNoStart) continue;
          int q = -1;
          for (int j = 0; j < C; ++j) {
            const uint32_t sj = st[uC + j];
            if (sj < p) q = max(q, (int)sj);    // kNoStart is above every position
          }
          if (q < 0) flags[1] = 1;
          else atomicMax(&b[q], (int)p);
        }
      }
    }
    __syncthreads();

    // per node: does it occur, what does it add to the duration; its outputs are held from p through b[p]
    int my_dur = 0;
    for (int round = 0; round < n; round += kUnroll * kNT) {
      const int base = round + tid;
      int2 sd[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) sd[u] = base + u * kNT < n ? G.size_dur[base + u * kNT] : make_int2(0, 0);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int v = base + u * kNT;
        if (v >= n) continue;
        int times = 0;
        for (int i = 0; i < C; ++i) {
          const uint32_t p = st[v * C + i];
          if (p == kNoStart) continue;
          ++times;
          atomicAdd(&a[p], sd[u].x);
          atomicAdd(&a[b[p] + 1], -sd[u].x);
        }
        if (times == 0) flags[1] = 1;
        my_dur += times * sd[u].y;
      }
    }
    if (my_dur) atomicAdd(&flags[2], my_dur);
    __syncthreads();
    const int peak = block_peak_of_running_sum(a, T, scratch, tid);

    if (tid == 0) {
      const bool valid = flags[1] == 0;
      out[cand] = moc_decode_result{valid ? 1 : 0, length, valid ? (int64_t)peak : 0, valid ? (int64_t)flags[2] : 0};
    }
    __syncthreads();
  }
}

// ---- the same for C <= 4, in four passes with a barrier behind each.
//
// 1. One lane per node: its starts go to an entry of the node (16 bits each, counted from 1, 0: not
//    computed) and the copy's name to the position it starts at, without atomics: two copies on one
//    position show as fewer occupied positions than active copies (Eq. (6)).
// 2. The occupied positions are counted, eight to a thread in one 16-byte read.  Behind this every wave knows
//    whether there is an order; a row without one is left here.
// 3. The names in order of position.  One lane per node walks the node's consumers (moc_slices.h) and keeps,
//    for every computation of the node in order, the last start that falls between it and the next one: that
//    is how long its output is held, known to one lane, without atomics or an array to meet in.  Two starts
//    at a time in 16-bit halves of a register.  Memory rises at the computation and falls behind the last
//    use (Eq. (4) by events).
// 4. The running sum's maximum.  Then the sequence is written out in 16-byte stores.
//
// Bound by HBM (295 MB read and written, 61 us at the rate of a copy), with the vector ALU 63 % and LDS 45 % busy
// beside it.  n = 2000, C = 2, 8192 candidates: 124 us with one lane per edge, the last use of a
// computation collected by atomic maxima (five passes, 824 vector and 114 LDS instructions per wave and
// candidate); 81 us now (480 and 69).  Without the walk the kernel takes 61 us, without storing the sequence 67,
// without anything else it does as long as with it.
// Rows without an order, as many: 70 us (59 where each of them was found by an atomic on its start, at a cost
// to the others; 81 with passes 2 and 3 in one, which is no quicker for the others); n = 1000, 4096 rows 18 us
// (18; 25), n = 7000, 1000 rows 30 (36; 63), n = 3000, C = 1, 4096 rows 34 (23; 49): a row's loads are asked for
// when the one before it is decided, and to ask earlier takes registers that the walk needs.

// The copies of a node as they lie in a candidate's row: aligned as their elements are, no more
// (the global loads of this chip take several words at any word boundary).
template <int CT>
struct alignas(4) CopyStarts {
  int32_t s[CT];
};
template <typename I>
struct __attribute__((packed)) FlagBytes {
  I x;
};
typedef int Words2 __attribute__((ext_vector_type(2)));
typedef int Words4 __attribute__((ext_vector_type(4)));
constexpr int kRawBuffer = 0x00020000;   // word 3 of a buffer descriptor: plain bytes, offsets checked against the size
constexpr int kDropped = 0x40000000;     // an offset beyond any buffer here
static_assert(sizeof(moc_decode_result) == 24, "stored as six words; peak and duration stay below 2^31");

constexpr int kRows = kHeldRows;

// Two 16-bit numbers in a register.
typedef short Halves __attribute__((ext_vector_type(2)));
typedef unsigned short UHalves __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Halves halves(uint32_t w) { return __builtin_bit_cast(Halves, w); }
__device__ __forceinline__ uint32_t word(Halves h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ uint32_t min_halves(uint32_t a, uint32_t b) {   // unsigned (written out: the compiler makes compares of some)
  uint32_t r;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t max_halves(uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_pk_max_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t lower_half(uint32_t w) {   // the smaller of the two
  uint32_t r;
  asm("v_min_u32_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1" : "=v"(r) : "v"(w));
  return r;
}
__device__ __forceinline__ uint32_t upper_half(uint32_t w) {   // the larger
  uint32_t r;
  asm("v_max_u32_sdwa %0, %1, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1" : "=v"(r) : "v"(w));
  return r;
}

// A node's starts as they lie in LDS, two to a word.
template <int CT>
struct NodeStarts {
  static constexpr int kWords = CT <= 2 ? 1 : 2;
  uint32_t w[kWords];
};
template <int CT>
__device__ __forceinline__ NodeStarts<CT> read_starts(uint32_t addr) {
  NodeStarts<CT> r;
  if constexpr (CT == 1) {
    r.w[0] = lds_read_u16(addr);
  } else if constexpr (CT == 2) {
    r.w[0] = lds_read(addr);
  } else {
    const uint2 x = lds_read2(addr);
    r.w[0] = x.x;
    r.w[1] = x.y;
  }
  return r;
}

// Adds to or takes from a word of LDS that several waves meet in.
__device__ __forceinline__ void raise(int32_t* at, int x) { __hip_atomic_fetch_add(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void lower(int32_t* at, int x) { __hip_atomic_fetch_sub(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

constexpr int kNoUse = 0xFFFF;          // first use of an output that is not used
constexpr uint32_t kNever = 0x7FFFu;   // start of a computation that does not happen: above every position

// What the starts of its consumers say about a node.
template <int CT>
struct Uses {
  uint32_t at[CT];     // the node's starts in rising order, kNever for those that are not computed
  uint32_t last[CT];   // last use of each, in two halves that are joined at the end
  uint32_t least;      // first use of any (0-based), in two halves
  __device__ __forceinline__ void begin(const NodeStarts<CT>& su) {
    uint32_t w[NodeStarts<CT>::kWords];
#pragma unroll
    for (int k = 0; k < NodeStarts<CT>::kWords; ++k)   // 0 -> kNever: 0 - 1 wraps to the highest number
      w[k] = word(halves(min_halves(word(halves(su.w[k]) - Halves{1, 1}), 0x7FFE7FFEu)) + Halves{1, 1});
    if constexpr (CT == 1) {
      at[0] = w[0] & 0xFFFFu;
    } else if constexpr (CT == 2) {
      at[0] = lower_half(w[0]);
      at[1] = upper_half(w[0]);
    } else {
      const uint32_t l0 = lower_half(w[0]), h0 = upper_half(w[0]), l1 = lower_half(w[1]), h1 = upper_half(w[1]);
      const uint32_t x = max(l0, l1), y = min(h0, h1);
      at[0] = min(l0, l1);
      at[1] = min(x, y);
      at[2] = max(x, y);
      if constexpr (CT == 4) at[3] = max(h0, h1);
    }
#pragma unroll
    for (int i = 0; i < CT; ++i) last[i] = at[i];
    least = 0xFFFFFFFFu;
  }
  __device__ __forceinline__ void use(const NodeStarts<CT>& sv) {   // 0: no use
#pragma unroll
    for (int k = 0; k < NodeStarts<CT>::kWords; ++k) {
      uint32_t rest = sv.w[k];
      least = min_halves(least, word(halves(rest) - Halves{1, 1}));
#pragma unroll
      for (int i = CT - 1; i > 0; --i) {   // the latest computation takes the uses behind it, the others go on
        uint32_t behind;
        asm("v_pk_sub_i16 %0, %1, %2 op_sel_hi:[0,1]" : "=v"(behind) : "v"(at[i]), "v"(sv.w[k]));
        behind = word(halves(behind) >> 15);
        last[i] = max_halves(last[i], rest & behind);
        rest &= ~behind;
      }
      last[0] = max_halves(last[0], rest);
    }
  }
};

// LOOP: more nodes than node_slots a lane or more positions than eight: the workgroup goes over them in
// rounds and reads the graph again for every candidate.  Otherwise what a lane needs of the graph stays in
// registers, and the starts and flags of the workgroup's next candidate are asked for while this one is
// still being worked on.
template <int CT, int NT, bool LOOP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8, 8)))
void decode_fixed_kernel(GraphView G, const uint32_t* __restrict__ slices, int64_t B, const int32_t* __restrict__ starts,
                         const uint8_t* __restrict__ active, moc_decode_result* __restrict__ out,
                         int32_t* __restrict__ out_seq, DfLayout lay) {
  extern __shared__ int32_t lds[];
  constexpr int SS = starts_stride(CT), NW = NT / kWave, R = LOOP ? 2 : 1, kSlots = node_slots(CT);
  char* const raw = reinterpret_cast<char*>(lds);   // at LDS address 0: [n + 1][SS] starts
  uint16_t* const pos = reinterpret_cast<uint16_t*>(raw + lay.pos_off);     // copy (+ 1) that starts at a position, 0: none
  uint16_t* const list = reinterpret_cast<uint16_t*>(raw + lay.list_off);   // the sequence, copies (+ 1), 0 behind its end
  int32_t* const a = reinterpret_cast<int32_t*>(raw + lay.a_off);           // memory differences
  int32_t* const told = reinterpret_cast<int32_t*>(raw + lay.told_off);     // by all waves: [0] copies computed beyond the positions taken, all candidates together; [2] is it not valid, [3] duration
  int32_t* const told_taken = told + (LOOP ? 4 : 4 + 2 * NW);               // per wave: positions taken
  // Per round and wave: sum and highest running sum.  LOOP: nobody asks for the starts any more when they are written,
  // and the wave that reads them is the one that writes these nodes' starts again.
  const auto sums = [&](int r, int w) { return reinterpret_cast<int2*>(LOOP ? raw + r * NT * 2 * SS : raw + lay.told_off + 16) + w; };
  static_assert(NW * 8 <= kWave * 2 * SS || !LOOP, "sums of a round in the starts of 64 nodes");
  const int tid = threadIdx.x;
  const int T = G.T, n = G.n;

  for (int x = 8 * tid; x < lay.T_pad; x += 8 * NT) {
    const int4 zero = make_int4(0, 0, 0, 0);
    *reinterpret_cast<int4*>(pos + x) = zero;
    *reinterpret_cast<int4*>(list + x) = zero;
    *reinterpret_cast<int4*>(a + x) = zero;
    *reinterpret_cast<int4*>(a + x + 4) = zero;
  }
  if (tid < SS) reinterpret_cast<uint16_t*>(lds)[n * SS + tid] = 0;   // node n is never computed
  if (tid < 4) told[tid] = 0;

  // The loads of a round of nodes are issued without conditions (lanes past the last node read
  // it again and drop what they get) and all of them before the first is looked at; a node's flags
  // stay as they arrive, in one register (three copies: two).  Loads under a condition, or flags put
  // together from several loads, end up one behind the other, each waiting for the one before.
  struct Round {
    int32_t s[kSlots][CT];
    uint32_t on[kSlots][CT == 3 ? 2 : 1];
    __device__ __forceinline__ lanemask active(int u, int i) const {
      return CT == 3 && i == 2 ? byte_ne_k(on[u][CT == 3 ? 1 : 0], 0, 0u) : byte_ne_k(on[u][0], i, 0u);
    }
  };
  // (the candidate's rows are scalar base addresses, a lane adds a 32-bit offset)
  auto request = [&](int64_t c, int round, int t, Round& r) {
    const char* const s_row = reinterpret_cast<const char*>(starts + c * T);
    const char* const a_row = reinterpret_cast<const char*>(active + c * T);
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const uint32_t off = (uint32_t)min(round + u * NT + t, n - 1) * CT;
      const CopyStarts<CT> sv = *reinterpret_cast<const CopyStarts<CT>*>(s_row + off * 4u);
#pragma unroll
      for (int i = 0; i < CT; ++i) r.s[u][i] = sv.s[i];
      if constexpr (CT == 1) r.on[u][0] = *reinterpret_cast<const uint8_t*>(a_row + off);
      else if constexpr (CT == 4) r.on[u][0] = reinterpret_cast<const FlagBytes<uint32_t>*>(a_row + off)->x;
      else r.on[u][0] = reinterpret_cast<const FlagBytes<uint16_t>*>(a_row + off)->x;
      if constexpr (CT == 3) r.on[u][1] = *reinterpret_cast<const uint8_t*>(a_row + off + 2);
    }
  };
  // A slice: where its rows of consumers begin and how many there are; the lane's node with its m_v, w_v.
  const int n_slices = (int)slices[0], n_apart = (int)slices[1];
  struct Slice {
    uint32_t rows;
    int count;
    uint32_t node;
    int size, dur;
  };
  auto open_slice = [&](int i, int lane) {
    Slice s;
    const uint32_t at = slices[2 + i];
    s.rows = at + kWave;
    s.count = (int)((slices[3 + i] - at) / kWave) - 1;
    s.node = slices[at + lane];
    const int2 sd = G.size_dur[min((int)s.node, n - 1)];
    s.size = sd.x;
    s.dur = sd.y;
    return s;
  };
  // The slices of a wave: the long ones come first, so every second round is dealt in reverse.
  auto slice_of = [](int u, int wave) { return u * NW + (u & 1 ? NW - 1 - wave : wave); };
  [[maybe_unused]] Round ahead;            // the workgroup's next candidate
  [[maybe_unused]] Slice mine[kSlots];
  [[maybe_unused]] uint32_t my_rows[kSlots][kRows];
  if constexpr (!LOOP) {
    request(blockIdx.x, 0, tid, ahead);   // the grid is not larger than the batch
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int i = slice_of(u, wave);
      mine[u] = Slice{0u, -1, 0u, 0, 0};
      if (i < n_slices) mine[u] = open_slice(i, lane);
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        my_rows[u][r] = 0;
        if (r < mine[u].count) my_rows[u][r] = slices[mine[u].rows + r * kWave + lane];
      }
    }
  }
  // Nothing is on its way into the loop: what it waits for is counted from its own operations alone.
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  __syncthreads();

  int beyond_before = 0;
  for (int64_t cand = blockIdx.x; cand < B; cand += gridDim.x) {
    // What derives from the thread index (row bounds, LDS addresses) is formed again for every
    // candidate: kept across candidates it takes registers that the next candidate's copies need.
    int t_ = tid;
    asm volatile("" : "+v"(t_));
    const int lane_ = t_ & (kWave - 1);
    const int wave_ = __builtin_amdgcn_readfirstlane(t_ / kWave);
    int32_t* const seq_row = out_seq ? out_seq + cand * T : nullptr;

    // ---- 1. who is computed where.  Predicates are lane masks; those of lanes past the last node are 0.
    int n_active = 0;           // copies computed, also where the start lies outside [0, T), Eq. (8)
    lanemask missing = 0;       // a node that is not computed
    auto lanes_in = [&](int round, int u) -> lanemask {   // the lanes that have a node in this slot
      const int left = n - (round + u * NT + wave_ * kWave);
      return left <= 0 ? 0 : left >= kWave ? ~(lanemask)0 : ((lanemask)1 << left) - 1;
    };
    auto place = [&](int round, const Round& r) {
#pragma unroll
      for (int u = 0; u < kSlots; ++u) {
        const lanemask in = lanes_in(round, u);
        if (in == 0) continue;
        const uint32_t v = (uint32_t)(round + u * NT + t_), name = v * CT + 1u;
        lanemask any = 0;
        uint32_t where[SS];   // the node's entry of the starts, written in one piece
#pragma unroll
        for (int i = 0; i < SS; ++i) where[i] = 0;
#pragma unroll
        for (int i = 0; i < CT; ++i) {
          const uint32_t at = (uint32_t)r.s[u][i];
          const lanemask on = r.active(u, i) & in, well = u_lt_k(at, (uint32_t)T), ok = on & well;
          n_active += count(on);
          any |= on;
          where[i] = pick(ok, at + 1u);
          lds_write16_lanes<0>(ok, (uint32_t)lay.pos_off + 2u * at, name + i);
        }
        missing |= in & ~any;
        if constexpr (SS == 1) lds_write16_lanes<0>(in, v * 2u, where[0]);
        else if constexpr (SS == 2) lds_write_lanes(in, v * 4u, where[0] | where[1] << 16);
        else if (lanes(in)) *reinterpret_cast<uint2*>(raw + v * 8u) = make_uint2(where[0] | where[1] << 16, where[2] | where[3] << 16);
      }
    };
    [[maybe_unused]] uint32_t more_rows[kRows];   // of the first slice, the longest; asked for before there is anything to wait for
    if constexpr (!LOOP) {
#pragma unroll
      for (int k = 0; k < kRows; ++k)
        more_rows[k] = slices[row_ahead(mine[0].rows, mine[0].count, kRows + k) + (uint32_t)lane_];
      place(0, ahead);
    } else {
      for (int round = 0; round < n; round += kSlots * NT) {
        Round now;
        request(cand, round, t_, now);
        __builtin_amdgcn_sched_barrier(0);
        place(round, now);
      }
    }
    wait_for_lds_writes();
    __syncthreads();

    // ---- 2. how many positions are taken; eight of them per thread and round
    int4 who[R];
    int taken = 0;   // those of the second round in the upper half
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int x = (r * NT + t_) * 8;
      who[r] = make_int4(0, 0, 0, 0);
      if (x < lay.T_pad) {
        who[r] = *reinterpret_cast<const int4*>(pos + x);
        *reinterpret_cast<int4*>(pos + x) = make_int4(0, 0, 0, 0);
      }
      const auto ones = [](int w) { return min_halves((uint32_t)w, 0x00010001u); };   // 1 in each half that is not 0
      const uint32_t c = ones(who[r].x) + ones(who[r].y) + ones(who[r].z) + ones(who[r].w);
      taken += (int)((c & 0xFFFFu) + (c >> 16)) << (16 * r);
    }
    const int upto = scan_sum(taken);
    const auto ask_for_next = [&] {   // (the last candidate asks for itself again)
      if constexpr (!LOOP) request(cand + gridDim.x < B ? cand + gridDim.x : cand, 0, t_, ahead);
    };
    const auto scan_row = [](int x) {
      x += lane_shift<0x111, 0xF>(x);
      x += lane_shift<0x112, 0xF>(x);
      x += lane_shift<0x114, 0xF>(x);
      x += lane_shift<0x118, 0xF>(x);
      return x;
    };
    if (lane_ == kWave - 1) {
      told_taken[wave_] = upto;
      raise(&told[0], n_active - ((upto & 0xFFFF) + (upto >> 16)));
    }
    __syncthreads();

    // ---- is there an order: lanes 0 .. NW - 1 hold one wave each
    const int beyond = __builtin_amdgcn_readfirstlane(told[0]);
    const int pairs = scan_row(lane_ < NW ? told_taken[lane_] : 0);
    const int total_taken = __builtin_amdgcn_readlane(pairs, NW - 1);
    const int taken_before = NW > 1 && wave_ > 0 ? __builtin_amdgcn_readlane(pairs, max(wave_ - 1, 0)) : 0;
    const int length = (total_taken & 0xFFFF) + (total_taken >> 16);
    // a start outside the domain, or two copies on one position: more copies than positions, no order
    const bool decodable = beyond == beyond_before;
    beyond_before = beyond;
    if (decodable) {
      // ---- 3. the names in order
      if (seq_row) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int before = (taken_before + upto - taken) >> (16 * r) & 0xFFFF;
          uint32_t at = (uint32_t)(before + (r ? total_taken & 0xFFFF : 0));
          const auto put_two = [&](uint32_t w) {
            const lanemask lo = low_ne_k(w, 0u), hi = high_ne_k(w, 0u);
            lds_write16_lanes<0>(lo, (uint32_t)lay.list_off + 2u * at, w);
            at = add_lanes(lo, at);
            lds_write16_lanes<1>(hi, (uint32_t)lay.list_off + 2u * at, w);
            at = add_lanes(hi, at);
          };
          put_two((uint32_t)who[r].x);
          put_two((uint32_t)who[r].y);
          put_two((uint32_t)who[r].z);
          put_two((uint32_t)who[r].w);
        }
      }
      // ---- and how long every output is held
      lanemask unserved = 0;
      int dur = 0;   // Eq. (1), this lane's nodes
      auto hold = [&](const Uses<CT>& uses, int size, int w) {
#pragma unroll
        for (int i = 0; i < CT; ++i)
          if (lanes(u_lt_k(uses.at[i], kNever))) {   // computed
            raise(&a[uses.at[i]], size);
            lower(&a[upper_half(uses.last[i]) + 1u], size);
            dur += w;
          }
      };
      auto two_uses = [&](Uses<CT>& uses, uint32_t row) {
        uint32_t lo, hi;   // taken apart here: moved out of the loop over the candidates the halves would take registers of their own
        asm volatile("v_and_b32 %0, 0xffff, %1" : "=v"(lo) : "v"(row));
        asm volatile("v_lshrrev_b32 %0, 16, %1" : "=v"(hi) : "v"(row));
        const NodeStarts<CT> x = read_starts<CT>(lo), y = read_starts<CT>(hi);
        uses.use(x);
        uses.use(y);
      };
      auto walk = [&](const Slice& s, const uint32_t* first_rows, const uint32_t* next_rows) {   // the first kRows, the kRows behind them, or null
        Uses<CT> uses;
        uses.begin(read_starts<CT>(s.node * (2u * SS)));
        int count = s.count, r = 0;
        asm volatile("" : "+s"(count));   // (compared here, not kept as a condition across the candidates)
        if (first_rows) {
#pragma unroll
          for (int k = 0; k < kRows; ++k)
            if (k < count) two_uses(uses, first_rows[k]);
          r = kRows;
        }
        if (next_rows) {
#pragma unroll
          for (int k = 0; k < kRows; ++k)
            if (kRows + k < count) two_uses(uses, next_rows[k]);
          r = 2 * kRows;
        }
        for (; r < count; r += kRows) {
          uint32_t row[kRows];
#pragma unroll
          for (int k = 0; k < kRows; ++k) row[k] = slices[s.rows + (uint32_t)(min(r + k, count - 1) * kWave + lane_)];
#pragma unroll
          for (int k = 0; k < kRows; ++k)
            if (k == 0 || r + k < count) two_uses(uses, row[k]);
        }
        unserved |= u_lt(lower_half(uses.least), uses.at[0]);
        hold(uses, s.size, s.dur);
      };
      if constexpr (!LOOP) {
#pragma unroll
        for (int u = 0; u < kSlots; ++u)
          if (mine[u].count >= 0) walk(mine[u], my_rows[u], u == 0 ? more_rows : nullptr);
      } else {
        for (int u = 0; u * NW < n_slices; ++u) {
          const int i = slice_of(u, wave_);
          if (i < n_slices) walk(open_slice(i, lane_), nullptr, nullptr);
        }
      }
      for (int i = wave_; i < n_apart; i += NW) {   // a node with very many consumers: all lanes of a wave
        const int v = (int)slices[3 + n_slices + i];
        Uses<CT> uses;
        uses.begin(read_starts<CT>((uint32_t)v * (2u * SS)));
        const int y1 = G.out_ptr[v + 1];
        for (int y = G.out_ptr[v]; y < y1; y += kWave)
          uses.use(read_starts<CT>((uint32_t)(y + lane_ < y1 ? G.out_idx[y + lane_] : n) * (2u * SS)));
        const int first = kNoUse - last_lane(scan_max(kNoUse - (int)lower_half(uses.least)));
        unserved |= (uint32_t)first < (uint32_t)__builtin_amdgcn_readfirstlane((int)uses.at[0]) ? 1 : 0;
#pragma unroll
        for (int k = 0; k < CT; ++k) uses.last[k] = (uint32_t)last_lane(scan_max((int)upper_half(uses.last[k])));
        if (lane_ == 0) {
          const int2 sd = G.size_dur[v];
#pragma unroll
          for (int k = 0; k < CT; ++k)
            if (uses.at[k] < kNever) {
              raise(&a[uses.at[k]], sd.x);
              lower(&a[uses.last[k] + 1u], sd.x);
              dur += sd.y;
            }
        }
      }
      dur = scan_sum(dur);
      if (lane_ == kWave - 1) raise(&told[3], dur);
      if ((missing | unserved) != 0 && lane_ == 0) told[2] = 1;
    }
    ask_for_next();
    if (decodable) {
      __syncthreads();

      // ---- 4. the peak of the running sum, eight positions per thread and round; the differences are left at zero
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int x = (r * NT + t_) * 8;
        int S = 0, P = 0;
        if (x < lay.T_pad) {
          const int4 lo = *reinterpret_cast<const int4*>(a + x), hi = *reinterpret_cast<const int4*>(a + x + 4);
          *reinterpret_cast<int4*>(a + x) = make_int4(0, 0, 0, 0);
          *reinterpret_cast<int4*>(a + x + 4) = make_int4(0, 0, 0, 0);
          S = lo.x; P = max(S, 0);
          S += lo.y; P = max(P, S);
          S += lo.z; P = max(P, S);
          S += lo.w; P = max(P, S);
          S += hi.x; P = max(P, S);
          S += hi.y; P = max(P, S);
          S += hi.z; P = max(P, S);
          S += hi.w; P = max(P, S);
        }
        combine_segments(S, P);
        if (lane_ == kWave - 1) *sums(r, wave_) = make_int2(S, P);   // the lane that holds the wave's
      }
      wait_for_lds_writes();
      __syncthreads();
    }

    // The sequence and the result.  Every wave issues the same stores, with lanes that have nothing to write
    // out of the buffer's range (such a store is dropped): a wave waits for its loads by the number of
    // memory operations behind them, and the loads that are on their way for the next candidate would
    // otherwise be waited for together with stores that may or may not have been issued.
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(seq_row, 0, seq_row ? 4 * T : 0, kRawBuffer);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int x = (r * NT + t_) * 8;
      int4 e = make_int4(0, 0, 0, 0);   // entries behind the sequence are 0 and become -1; so do all if there is none
      if (seq_row && decodable && x < length) {
        e = *reinterpret_cast<const int4*>(list + x);
        *reinterpret_cast<int4*>(list + x) = make_int4(0, 0, 0, 0);
      }
      const auto node_of = [](uint32_t name) -> int {
        if constexpr (CT == 3) return (int)((name + 2u) / 3u) - 1;
        else return ((int)name - 1) >> (CT / 2);
      };
      const uint32_t w[4] = {(uint32_t)e.x, (uint32_t)e.y, (uint32_t)e.z, (uint32_t)e.w};
      Words4 four[2];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        four[j / 2][2 * (j & 1)] = node_of(w[j] & 0xFFFFu);
        four[j / 2][2 * (j & 1) + 1] = node_of(w[j] >> 16);
      }
      const int off = x + 8 <= T ? 4 * x : kDropped;
      __builtin_amdgcn_raw_buffer_store_b128(four[0], rows, off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(four[1], rows, off, 16, 0);
      if ((T & 7) != 0 && seq_row) {   // the last thread of a row that is not a multiple of eight
#pragma unroll
        for (int j = 0; j < 7; ++j)
          if (x + 8 > T && x + j < T) seq_row[x + j] = four[j / 4][j & 3];
      }
    }
    // No barrier behind this: what is read here is written again behind the next candidate's second.
    int2 segment = make_int2(0, 0);
    int total_dur = 0;
    bool valid = false;
    if (wave_ == 0 && decodable) {
      if (lane_ < R * NW) segment = *sums(lane_ / NW, lane_ % NW);
      combine_segments(segment.x, segment.y);
      const int2 about = *reinterpret_cast<const int2*>(told + 2);   // faults, duration
      valid = __builtin_amdgcn_readfirstlane(about.x) == 0;
      total_dur = __builtin_amdgcn_readfirstlane(about.y);
      int zero = 0;
      asm volatile("" : "+v"(zero));   // (a constant here is kept in registers across the candidates)
      lds_write_lanes(1, (uint32_t)lay.told_off + 8u, (uint32_t)zero);
      lds_write_lanes(1, (uint32_t)lay.told_off + 12u, (uint32_t)zero);
    }
    const auto result = __builtin_amdgcn_make_buffer_rsrc(out + cand, 0, (int)sizeof(moc_decode_result), kRawBuffer);
    const int off = wave_ == 0 && lane_ == kWave - 1 ? 0 : kDropped;
    __builtin_amdgcn_raw_buffer_store_b128(Words4{decodable ? (valid ? 1 : 0) : -1, decodable ? length : 0, valid ? segment.y : 0, 0},
                                           result, off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b64(Words2{valid ? total_dur : 0, 0}, result, off, 16, 0);
  }
}

using DfKernel = void (*)(GraphView, const uint32_t*, int64_t, const int32_t*, const uint8_t*, moc_decode_result*, int32_t*, DfLayout);

template <int CT>
DfKernel pick_fixed(int nt, bool loop) {
  if (loop) return decode_fixed_kernel<CT, 1024, true>;
  switch (nt) {
    case 64: return decode_fixed_kernel<CT, 64, false>;
    case 128: return decode_fixed_kernel<CT, 128, false>;
    case 256: return decode_fixed_kernel<CT, 256, false>;
    case 512: return decode_fixed_kernel<CT, 512, false>;
    default: return decode_fixed_kernel<CT, 1024, false>;
  }
}

}  // namespace

extern "C" int moc_decode_batch(const moc_graph* g, int64_t B, const int32_t* starts, const uint8_t* active,
                                moc_decode_result* out, int32_t* out_seq, void* hip_stream) {
  if (!g || B < 0) return MOC_EINVAL;
  if (B == 0) return MOC_OK;
  if (!starts || !active || !out) return MOC_EINVAL;
  if (((uintptr_t)starts & 3) || ((uintptr_t)out & 7) || ((uintptr_t)out_seq & 3)) return MOC_EINVAL;
  int dev = -1;
  MOC_HIP(hipGetDevice(&dev));
  if (dev != g->device) return MOC_EDEVICE;
  const GraphView& v = g->view;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (!decode_fits(v.n, v.C, g->max_lds)) return MOC_EOVERFLOW;
  const auto resident = [&](const void* kern, int nt, int bytes, bool no_static_lds, unsigned* grid) -> int {
    int per_cu = 0;
    if (const int rc = moc_kernel_occupancy(g, kern, nt, bytes, no_static_lds, &per_cu)) return rc;
    *grid = (unsigned)std::min<int64_t>(B, (int64_t)per_cu * g->num_cu);
    return MOC_OK;
  };
  if (g->slices) {   // C <= 4
    const DecodeShape shape = decode_shape(v.n, v.C, B, g->num_cu);
    const int nt = shape.nt;
    const DfLayout lay = shape.lay;
    if (lay.bytes > g->max_lds) return MOC_EOVERFLOW;   // (fits wherever decode_fits holds)
    DfKernel kern = nullptr;
    switch (v.C) {
      case 1: kern = pick_fixed<1>(nt, shape.loop); break;
      case 2: kern = pick_fixed<2>(nt, shape.loop); break;
      case 3: kern = pick_fixed<3>(nt, shape.loop); break;
      default: kern = pick_fixed<4>(nt, shape.loop); break;
    }
    unsigned grid = 0;
    if (const int rc = resident(reinterpret_cast<const void*>(kern), nt, lay.bytes, true, &grid)) return rc;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lay.bytes, stream, v, g->slices, B, starts, active, out, out_seq, lay);
    MOC_HIP(hipGetLastError());
    return MOC_OK;
  }
  const DcLayout any = dc_layout(v.n, v.C);
  unsigned grid = 0;
  if (const int rc = resident(reinterpret_cast<const void*>(decode_kernel), kNT, any.bytes, false, &grid)) return rc;
  hipLaunchKernelGGL(decode_kernel, dim3(grid), dim3(kNT), any.bytes, stream, v, B, starts, active, out, out_seq, any);
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}
