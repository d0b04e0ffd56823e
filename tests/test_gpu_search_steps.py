"""GPU parity of the searches that take a candidate through all its steps in one launch, where
their kernels can go wrong: edges of the 64-copy chunks, of the blocks of 8 positions and of the
rows of 256, one to five copies per node, lists cut at K, shared starts, steps that run out."""
import numpy as np
import pytest

import oracle
from test_gpu_cuts import schedules, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moc():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2304_14463_amd import moccasin
    moccasin.lib()
    return moccasin


def random_graph(rng, n):
    from paper_2304_14463_amd.inputs import graph_from_edges
    edges = []
    for v in range(1, n):
        for u in rng.integers(max(0, v - 12), v, size=rng.integers(1, 4)):
            edges.append((int(u), v))        # duplicates stay
    return graph_from_edges(n, sorted(edges), rng.integers(0, 50, n), rng.integers(1, 9, n))


def recomputed(rng, g, C, B):
    """Schedules in which most nodes are computed several times, every output kept to the next
    computation of its node: full of merges, violation-free; then rows with one copy moved onto
    another's start (a merge of that copy mends it), and rows of stray copies."""
    n, T = g.n, g.n * C
    s, e, a = schedules(rng, g, C, B, wild=True)
    for b in range(0, B, 3):
        pos = np.arange(n) * C
        last = pos.copy()
        for v in range(n):
            for u in g.in_idx[g.in_ptr[v]:g.in_ptr[v + 1]]:
                last[u] = max(last[u], pos[v] + C - 1)
        last = np.minimum(last + C - 1, T - 1)
        for v in range(n):
            live = [i for i in range(C) if i == 0 or rng.random() < 0.7]
            for i in range(C):
                k = v * C + i
                a[b, k] = 1 if i in live else 0
                s[b, k] = pos[v] + i
                later = [j for j in live if j > i]
                e[b, k] = pos[v] + later[0] if later else max(last[v], pos[v] + i)
        if (b // 3) % 2 and n > 1 and C > 1:
            k = int(rng.integers(1, n)) * C + C - 1
            a[b, k], s[b, k] = 1, s[b, k - C]
            e[b, k] = max(e[b, k], s[b, k])
    return s, e, a


@pytest.mark.parametrize("n,C,K", [(1, 1, 4), (3, 2, 1), (4, 2, 8), (16, 2, 5), (32, 2, 64), (33, 2, 64), (64, 4, 300), (85, 3, 200),
                                   (128, 2, 64), (129, 2, 3), (51, 5, 64), (256, 2, 400), (300, 4, 64), (2100, 4, 32)])
def test_merges_follow_the_oracle(moc, n, C, K):
    """Second phase alone: counts and rows after it are the oracle's, field by field."""
    rng = np.random.default_rng(97 * n + 5 * C + K)
    g = random_graph(rng, n)
    B, steps = (12, 9) if n < 1000 else (3, 2)
    s, e, a = recomputed(rng, g, C, B)
    peaks = oracle.evaluate(g, 0, C, s, e, a)[:, 0]
    budget = int(np.median(peaks))
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(s, e, a)
    cuts, merges = moc.moc_search_two_phase(gh, ds, de, da, 0, steps, K)
    merges, gs, ge, ga = merges.cpu().numpy(), ds.cpu().numpy(), de.cpu().numpy(), da.cpu().numpy()
    assert (cuts.cpu().numpy() == 0).all()
    for b in range(B):
        _, k, ws, we, wa = oracle.search_two_phase(g, budget, C, s[b], e[b], a[b], 0, steps, K)
        assert merges[b] == k, (b, merges[b], k)
        assert (ga[b] == wa).all() and (gs[b] == ws).all() and (ge[b] == we).all(), b
    assert C == 1 or n < 4 or merges.max() > 0
    gh.free()
