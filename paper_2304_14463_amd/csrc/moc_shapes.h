// Rules by which the host picks a kernel's shape for a graph and a batch: plain C++, so that they can
// be checked over all sizes without a GPU.
#pragma once

// ------------------------------------------------------------------ moc_eval_batch_staged
constexpr int kStagedThreads = 512;

// Nodes per lane of the kernel that holds the copies of a lane's nodes in registers (built for 1, 2,
// 4 and 8, as long as a lane has at most 16 copies), 0: the kernel for any size.  The node loops and
// the scan over the stages of the former cover kStagedThreads times this many nodes and no more.
constexpr int staged_nodes_per_lane(int n, int C) {
  int u = 1;
  while (u * kStagedThreads < n) u *= 2;
  return C <= 4 && u <= 8 && u * C <= 16 ? u : 0;
}
