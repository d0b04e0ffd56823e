"""moc_eval_batch with five copies a node in registers: sizes on either side of its thread counts and of the LDS limit, any
alignment, every copy live or few, against the oracle."""
import numpy as np
import pytest

from helpers import assert_results_equal, oracle_eval_parallel
from test_gpu_neighbours import moc, random_candidates, to_dev  # noqa: F401  (moc: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,degree,B", [(1, 0, 9), (2, 1, 9), (3, 1, 70), (64, 2, 600), (65, 3, 70), (191, 2, 3000), (192, 1, 40), (193, 3, 40), (385, 3, 40), (400, 9, 40),
                                        (769, 2, 2000), (1537, 2, 40), (2960, 3, 300), (3343, 3, 12), (3344, 3, 12), (300, 40, 12),
                                        (1500, 10, 12), (1500, 13, 12), (3300, 5, 12), (1500, 14, 12)])
def test_five_copies(moc, n, degree, B):  # noqa: F811
    import torch
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(n * 31 + degree)
    g = graph_from_edges(n, sorted({(int(u), v) for v in range(1, n) for u in rng.integers(max(0, v - 60), v, size=degree)}), rng.integers(0, 60, n), rng.integers(0, 9, n))
    T, C = 5 * n, 5
    rows = min(B, 40)
    s, e, a = random_candidates(rng, rows, T, T, wild=True)
    plain = slice(0, rows // 2)      # the plain schedule, some with further copies behind the first, some with shifted starts
    s[plain], e[plain], a[plain] = 0, 0, 0
    s[plain, ::C] = np.arange(n) * C
    e[plain, ::C] = np.minimum(s[plain, ::C] + C * rng.integers(0, 61, (rows // 2, n)), T - 1)
    a[plain, ::C] = 1
    for i in range(1, C):
        more = rng.random((rows // 2, n)) < np.linspace(0, 1, rows // 2)[:, None]
        a[plain, i::C] = more
        s[plain, i::C] = np.arange(n) * C + i
        e[plain, i::C] = np.minimum(s[plain, i::C] + rng.integers(0, 40, (rows // 2, n)), T - 1)
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, int(g.size.sum()), C)
    pick = np.arange(B) % rows
    ref = oracle_eval_parallel(g, int(g.size.sum()), C, s, e, a)
    assert_results_equal(moc.results_to_numpy(moc.moc_eval_batch(gh, *to_dev(s[pick], e[pick], a[pick]))), ref[pick], f"n={n}")
    shifted = []
    for x in to_dev(s, e, a):        # bases that are aligned to an element only
        room = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
        room[1:] = x.reshape(-1)
        shifted.append(room[1:].view(rows, T))
    assert_results_equal(moc.results_to_numpy(moc.moc_eval_batch(gh, *shifted)), ref, f"n={n}, shifted")
    out = torch.empty((rows, 24), dtype=torch.uint8, device="cuda")
    assert_results_equal(moc.results_to_numpy(moc.moc_eval_batch_noalloc(gh, *to_dev(s, e, a), out)), ref, f"n={n}, noalloc")
    gh.free()
