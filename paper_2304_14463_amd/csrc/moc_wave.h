// Wave scans by the lane shifts of the vector ALU.
#pragma once

#include "moc_internal.h"

namespace {

// The value of the lane CTRL names (a lane shift of the vector ALU), 0 where that lane does not
// exist or the row is not in ROWS.
template <int CTRL, int ROWS>
__device__ __forceinline__ int lane_shift(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, true); }

// Inclusive scans over the 64 lanes: inside rows of 16 by shifts of 1, 2, 4, 8, then lane 15 of
// rows 0 and 2 goes to rows 1 and 3, then lane 31 to rows 2 and 3.  Values of the maximum >= 0.
__device__ __forceinline__ int scan_sum(int x) {
  x += lane_shift<0x111, 0xF>(x);   // row_shr:1
  x += lane_shift<0x112, 0xF>(x);   // row_shr:2
  x += lane_shift<0x114, 0xF>(x);   // row_shr:4
  x += lane_shift<0x118, 0xF>(x);   // row_shr:8
  x += lane_shift<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
  x += lane_shift<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
  return x;
}
__device__ __forceinline__ int scan_max(int x) {
  x = max(x, lane_shift<0x111, 0xF>(x));
  x = max(x, lane_shift<0x112, 0xF>(x));
  x = max(x, lane_shift<0x114, 0xF>(x));
  x = max(x, lane_shift<0x118, 0xF>(x));
  x = max(x, lane_shift<0x142, 0xA>(x));
  x = max(x, lane_shift<0x143, 0xC>(x));
  return x;
}
__device__ __forceinline__ unsigned long long scan_max64(unsigned long long x) {
  const auto step = [&](int lo, int hi) {
    const unsigned long long o = (unsigned long long)(uint32_t)hi << 32 | (uint32_t)lo;
    x = o > x ? o : x;
  };
  step(lane_shift<0x111, 0xF>((int)x), lane_shift<0x111, 0xF>((int)(x >> 32)));
  step(lane_shift<0x112, 0xF>((int)x), lane_shift<0x112, 0xF>((int)(x >> 32)));
  step(lane_shift<0x114, 0xF>((int)x), lane_shift<0x114, 0xF>((int)(x >> 32)));
  step(lane_shift<0x118, 0xF>((int)x), lane_shift<0x118, 0xF>((int)(x >> 32)));
  step(lane_shift<0x142, 0xA>((int)x), lane_shift<0x142, 0xA>((int)(x >> 32)));
  step(lane_shift<0x143, 0xC>((int)x), lane_shift<0x143, 0xC>((int)(x >> 32)));
  return x;
}
__device__ __forceinline__ int last_lane(int x) { return __builtin_amdgcn_readlane(x, kWave - 1); }

// (sum, max prefix >= 0) of consecutive segments, one per lane, combined in lane order: each lane takes
// in the lanes before it (a lane with no source gets (0, 0), which changes nothing), the last lane ends
// with the whole wave.
template <int CTRL, int ROWS>
__device__ __forceinline__ void combine_earlier(int& S, int& P) {
  const int Se = lane_shift<CTRL, ROWS>(S), Pe = lane_shift<CTRL, ROWS>(P);
  P = max(Pe, Se + P);
  S = Se + S;
}
__device__ __forceinline__ void combine_segments(int& S, int& P) {
  combine_earlier<0x111, 0xF>(S, P);
  combine_earlier<0x112, 0xF>(S, P);
  combine_earlier<0x114, 0xF>(S, P);
  combine_earlier<0x118, 0xF>(S, P);
  combine_earlier<0x142, 0xA>(S, P);
  combine_earlier<0x143, 0xC>(S, P);
}

// The same over the first N <= 16 lanes, the others' values of no use.
template <int N>
__device__ __forceinline__ int scan_sum_first(int x) {
  if constexpr (N > 1) x += lane_shift<0x111, 0xF>(x);
  if constexpr (N > 2) x += lane_shift<0x112, 0xF>(x);
  if constexpr (N > 4) x += lane_shift<0x114, 0xF>(x);
  if constexpr (N > 8) x += lane_shift<0x118, 0xF>(x);
  return x;
}
template <int N>
__device__ __forceinline__ void combine_first(int& S, int& P) {
  if constexpr (N > 1) combine_earlier<0x111, 0xF>(S, P);
  if constexpr (N > 2) combine_earlier<0x112, 0xF>(S, P);
  if constexpr (N > 4) combine_earlier<0x114, 0xF>(S, P);
  if constexpr (N > 8) combine_earlier<0x118, 0xF>(S, P);
}

}  // namespace
