"""Merges with 512 threads (one walker to a compute unit, T > 900) against 256 (more walkers), walker by walker."""
import numpy as np
import pytest

from test_gpu_two_phase import moc  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,C,K", [(451, 2, 64), (500, 3, 5), (901, 1, 8), (300, 4, 100), (1100, 2, 64)])
def test_merges_do_not_depend_on_the_threads(moc, n, C, K):  # noqa: F811
    import torch
    from paper_2304_14463_amd.inputs import DeviceWorkload, graphs, workload_from_graph
    g = graphs.graph_from_edges(n, graphs.layered_dag_edges(n, n, max(4, n // 22), 1, 5, True, False, 3 * n),
                                graphs.lognormal_sizes(n, n, 5.0, 1.0), graphs.uniform_ints(n, graphs.S_DUR, n, 1, 200))
    w = workload_from_graph("merges", n, g, C, 128, 130)
    rows = DeviceWorkload(w).candidates(0, 40)
    gh = moc.moc_graph_upload(g.n, g.in_ptr, g.in_idx, g.size, g.dur, w.budget, C)
    few, many = [x.clone() for x in rows], [x.repeat(20, 1).contiguous() for x in rows]   # 40 and 800 walkers
    got = moc.moc_search_two_phase(gh, *few, 6, 20, K)
    want = moc.moc_search_two_phase(gh, *many, 6, 20, K)
    for x, y in zip(few + list(got), many + list(want)):
        assert torch.equal(x, y[:40])
    assert C == 1 or int(got[1].max()) > 0
    gh.free()
