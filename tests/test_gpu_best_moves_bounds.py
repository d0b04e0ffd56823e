"""The best single-field move of bases whose fields nearly all share the same bounds, against the kernel of the table."""
import numpy as np
import pytest

from test_gpu_best_moves import graph
from test_gpu_neighbours import gpu_neighbours, moc  # noqa: F401  (moc: fixture)

pytestmark = pytest.mark.gpu


def same_best(moc, g, C, R, s, e, a):  # noqa: F811
    gh = moc.moc_graph_upload(g.n, g.in_ptr, g.in_idx, g.size, g.dur, int(g.size.sum()) // 3, C)
    _, want = gpu_neighbours(moc, gh, s, e, a, R)
    _, got = gpu_neighbours(moc, gh, s, e, a, R, moves=False)
    bad = [b for b in range(len(s)) if got[b].tobytes() != want[b].tobytes()]
    assert not bad, (bad[:5], got[bad[0]], want[bad[0]])
    gh.free()


# every output kept to the end of the schedule: no violations, and every end is one that lowers the peak, by its node's
# size or by less where another position comes to be the highest
@pytest.mark.parametrize("n,C,R,sizes", [(60, 2, 8, "any"), (300, 1, 1, "any"), (300, 2, 9, "equal"), (300, 3, 32, "few"), (700, 2, 4, "zero"), (1100, 2, 16, "any"), (50, 5, 3, "few")])
def test_outputs_kept_to_the_end(moc, n, C, R, sizes):  # noqa: F811
    rng = np.random.default_rng(n + C + R)
    g = graph(rng, n, 2, size_hi=1 if sizes == "zero" else 1000)
    if sizes in ("equal", "few"):
        g.size[:] = 7 if sizes == "equal" else rng.choice([0, 5, 5, 6], n)
    B, T = 12, n * C
    s, e, a = (np.zeros((B, T), t) for t in (np.int32, np.int32, np.uint8))
    s[:, ::C] = np.arange(n) * C
    e[:, ::C] = T - 1
    a[:, ::C] = 1
    for b in range(1, B):
        e[b, ::C] -= rng.integers(0, 2 * b, n, dtype=np.int32)      # ends on either side of the peak's positions
    e = np.maximum(e, s)
    same_best(moc, g, C, R, s, e, a)
