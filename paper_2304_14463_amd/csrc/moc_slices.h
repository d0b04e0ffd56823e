// The consumers of every node as the decode kernel walks them: plain C++, so that it can be checked
// without a GPU.
//
// A lane takes a node and looks at the starts of its consumers one after the other, so the nodes of a
// wave should have the same number of them: nodes in order of falling out-degree, 64 to a slice.  A slice
// is stored by rows of 64 words, one word a lane: row 0 the nodes, each further row two consumers per
// lane (low and high half) as byte offsets of their starts.  Lanes and halves without one hold node n,
// which is never computed.  Nodes with very many consumers are listed apart: a wave takes one of them with
// all its lanes.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

constexpr int kSliceLanes = 64, kSliceDegree = 32;
constexpr int kHeldRows = 2;   // of a slice that the kernel keeps in registers
constexpr int starts_stride(int C) { return C == 3 ? 4 : C; }   // 16-bit entries of a node's starts in LDS

// Nodes with more consumers than this are listed apart.  Apart, a node takes a wave as long as 6.5 consumers take
// it in a slice (and 2.1 for every 64 consumers more), but the wave has nothing else to do; in a slice it takes
// its own number and 63 others with it, and the waves wait for the one with the longest.  So: of some limits
// the one under which the slowest of `waves` waves ends first.  Microseconds with a limit of 32 / 64 / 128 /
// 256 / none (one lane per edge): about 40 consumers each, n = 1000, C = 2, 4096 candidates 502 / 72 / 72 / 72 /
// 72 (145); about 100, 2048 candidates 345 / 330 / 76 / 76 / 76 (153); 20 nodes of 200, 4096 candidates 41 /
// 51 / 65 / 73 / 74 (44); n = 2000, 40 of 1000 111 / 123 / 146 / 231 / 488 (128); falling as 1000 / rank^0.7
// 148 / 111 / 121 / 180 / 430 (143).
inline int slice_degree(int n, int waves, const int32_t* out_ptr) {
  std::vector<int> d(n);
  for (int v = 0; v < n; ++v) d[v] = out_ptr[v + 1] - out_ptr[v];
  if (*std::max_element(d.begin(), d.end()) <= kSliceDegree) return kSliceDegree;
  std::sort(d.begin(), d.end(), [](int a, int b) { return a > b; });
  int best = kSliceDegree;
  double best_time = -1;
  for (int limit = kSliceDegree;; limit += limit / 4) {
    double all = 0, longest = 0;
    int k = 0;
    for (; k < n && d[k] > limit; ++k) all += 6.5 + 2.1 * ((d[k] - 1) / kSliceLanes);
    if (k < n) longest = d[k];
    for (int i = k; i < n; i += kSliceLanes) all += d[i];
    const double time = std::max(longest, all / waves);
    if (best_time < 0 || time < best_time) best_time = time, best = limit;
    if (k == 0) return best;
  }
}

// word 0: slices, word 1: nodes listed apart; then the word at which each slice begins and the one behind
// the last, the nodes listed apart, the slices.  Empty if the byte offsets need more than 16 bits.
inline std::vector<uint32_t> out_slices(int n, int C, const int32_t* out_ptr, const int32_t* out_idx, int degree = kSliceDegree) {
  if (C > 4 || (int64_t)n * 2 * starts_stride(C) > 0xFFFF) return {};
  std::vector<int32_t> order, apart;
  for (int v = 0; v < n; ++v) (out_ptr[v + 1] - out_ptr[v] > degree ? apart : order).push_back(v);
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return out_ptr[a + 1] - out_ptr[a] > out_ptr[b + 1] - out_ptr[b]; });
  const int slices = ((int)order.size() + kSliceLanes - 1) / kSliceLanes;
  const uint32_t bytes = 2u * (uint32_t)starts_stride(C), none = bytes * (uint32_t)n;
  std::vector<uint32_t> w(2 + slices + 1 + apart.size());
  w[0] = (uint32_t)slices;
  w[1] = (uint32_t)apart.size();
  for (size_t i = 0; i < apart.size(); ++i) w[2 + slices + 1 + i] = (uint32_t)apart[i];
  for (int s = 0; s < slices; ++s) {
    const size_t at = w.size();
    w[2 + s] = (uint32_t)at;
    const int first = order[(size_t)s * kSliceLanes], rows = (out_ptr[first + 1] - out_ptr[first] + 1) / 2;
    w.resize(at + (size_t)(1 + rows) * kSliceLanes, none | none << 16);
    for (int l = 0; l < kSliceLanes; ++l) {
      const size_t i = (size_t)s * kSliceLanes + l;
      w[at + l] = i < order.size() ? (uint32_t)order[i] : (uint32_t)n;
      if (i >= order.size()) continue;
      const int v = order[i];
      for (int y = out_ptr[v], k = 0; y < out_ptr[v + 1]; ++y, ++k) {
        uint32_t& word = w[at + (size_t)(1 + k / 2) * kSliceLanes + l];
        const uint32_t c = bytes * (uint32_t)out_idx[y];
        word = k & 1 ? (word & 0xFFFFu) | c << 16 : (word & 0xFFFF0000u) | c;
      }
    }
  }
  w[2 + slices] = (uint32_t)w.size();
  return w;
}

// The list as the kernel is given it, a row longer: the rows behind the kHeldRows of a wave's first slice are
// asked for whether there are any or not.  (With the index kept inside the list instead the kernel holds
// more in scalar registers than there are: 31 of them spilled instead of 21.)
inline std::vector<uint32_t> slices_for_kernel(int n, int C, int waves, const int32_t* out_ptr, const int32_t* out_idx) {
  std::vector<uint32_t> w = out_slices(n, C, out_ptr, out_idx, slice_degree(n, waves, out_ptr));
  if (!w.empty()) w.resize(w.size() + kSliceLanes);
  return w;
}
// Where row r of a slice begins for a wave that reads it so: its last row, the row behind it if it has none;
// (0, -1): no slice.
constexpr uint32_t row_ahead(uint32_t rows, int count, int r) {
  const int row = r < count - 1 ? r : count - 1;
  return rows + (uint32_t)((row > 0 ? row : 0) * kSliceLanes);
}
