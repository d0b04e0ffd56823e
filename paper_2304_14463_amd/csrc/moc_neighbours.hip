// moc_eval_neighbours and moc_search_moves: arguments, and the choice of a kernel.  The table of scores comes from
// moc_neighbours_table.hip; the best move alone and the descent from moc_best_moves.h, which does not score every
// move.
#include <algorithm>

#include "moc_best_moves.h"

namespace {

using BestKernel = void (*)(GraphView, int64_t, const int32_t*, const int32_t*, const uint8_t*, int, moc_best_move*, MoveSteps, BmLayout);

template <int NT, bool LOOP, bool SEARCH>
BestKernel pick_best(int C) {
  switch (C) {
    case 1: return best_neighbours_kernel<NT, LOOP, 1, SEARCH, !SEARCH>;
    case 2: return best_neighbours_kernel<NT, LOOP, 2, SEARCH, !SEARCH>;
    case 3: return best_neighbours_kernel<NT, LOOP, 3, SEARCH, !SEARCH>;
    case 4: return best_neighbours_kernel<NT, LOOP, 4, SEARCH, !SEARCH>;
    default: return best_neighbours_kernel<NT, LOOP, 0, SEARCH, !SEARCH>;   // C read at run time
  }
}
template <bool SEARCH>
BestKernel pick_best(int nt, bool loop, int C) {
  switch (nt) {
    case 256: return pick_best<256, false, SEARCH>(C);
    case 512: return loop ? pick_best<512, true, SEARCH>(C) : pick_best<512, false, SEARCH>(C);
    default: return pick_best<1024, true, SEARCH>(C);
  }
}

// One launch over B bases: the best move, or (search) the walkers' whole descents.
int queue_best(const moc_graph* g, int64_t B, const int32_t* starts, const int32_t* ends, const uint8_t* active, int32_t R,
               moc_best_move* out_best, const MoveSteps& search, hipStream_t stream) {
  const int T = g->view.T, nt = best_threads(T, B, g->num_cu, g->max_lds);
  const BmLayout lay = bm_layout(T, nt);
  const bool loop = T > 4 * nt;
  const BestKernel kern = search.steps ? pick_best<true>(nt, loop, g->view.C) : pick_best<false>(nt, loop, g->view.C);
  int per_cu = 0;
  if (const int rc = moc_kernel_occupancy(g, reinterpret_cast<const void*>(kern), nt, lay.bytes, false, &per_cu)) return rc;
  const int64_t resident = (int64_t)per_cu * g->num_cu;
  const unsigned grid = (unsigned)(B < resident ? B : resident);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lay.bytes, stream, g->view, B, starts, ends, active, R, out_best, search, lay);
  return MOC_OK;
}

// What both calls refuse about the graph: another device, an edge (v,v), a T too large for LDS or for 32-bit offsets.
int check_neighbours(const moc_graph* g, int32_t R) {
  int dev = -1;
  MOC_HIP(hipGetDevice(&dev));
  if (dev != g->device) return MOC_EDEVICE;
  if (g->has_self_loop) return MOC_EINVAL;
  if (!neighbours_fit(g->view.T, g->max_lds)) return MOC_EOVERFLOW;
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
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (const int rc = out_moves ? moc_queue_neighbour_table(g, B, starts, ends, active, R, out_moves, out_best, stream)
                               : queue_best(g, B, starts, ends, active, R, out_best, MoveSteps{}, stream))
    return rc;
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

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
  // One launch, a workgroup to a walker, which stays in LDS from its first step to its last.  (One launch a step,
  // every walker staged again: C = 2, n = 442, R = 8, 256 walkers, 16 steps 191 us, now 80; n = 1000, R = 4, 32 walkers, 8 steps
  // 154, now 70; 1024 walkers 351, now 142.)
  if (const int rc = queue_best(g, B, starts, ends, active, R, work_best, MoveSteps{starts, ends, out_steps, max_steps}, stream)) return rc;
  MOC_HIP(hipGetLastError());
  return MOC_OK;
}

