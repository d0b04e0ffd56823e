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


# rows in which most fields have much the same bound, and rows at the ends of the domain, where a field's moves are cut off
@pytest.mark.parametrize("kind", ["anywhere", "short", "at the ends", "all at 0", "none well formed", "in any order"])
@pytest.mark.parametrize("n,C,R,per_node", [(60, 2, 8, 2), (442, 2, 8, 2), (300, 3, 1, 3), (250, 4, 32, 2), (1100, 2, 2, 2), (50, 5, 16, 20)])
def test_bases_far_from_a_schedule(moc, n, C, R, per_node, kind):  # noqa: F811
    rng = np.random.default_rng(n + C + R + len(kind))
    g = graph(rng, n, per_node, size_hi=4 if n % 100 else 1000)
    B, T = 14, n * C
    s, e = (rng.integers(0, T, (B, T), dtype=np.int32) for _ in range(2))
    s, e, a = np.minimum(s, e), np.maximum(s, e), (rng.random((B, T)) < 0.8).astype(np.uint8)
    if kind == "short":
        e = np.minimum(s + rng.integers(0, 1 + T // 20, (B, T), dtype=np.int32), T - 1)
    elif kind == "at the ends":
        s = rng.choice([-1, 0, 0, 1, T - 2, T - 1], (B, T)).astype(np.int32)
        e = np.minimum(s + rng.choice([0, 1, R, T], (B, T)).astype(np.int32), T - 1 + (rng.random((B, T)) < 0.1))
    elif kind == "all at 0":
        s[:], e[:] = 0, np.arange(B, dtype=np.int32)[:, None] // 2
    elif kind == "none well formed":
        s, e = np.maximum(s, 1), np.minimum(s, T - 2) - rng.integers(1, 2 * R + 1, (B, T), dtype=np.int32)
    elif kind == "in any order":
        a[:], a[:, ::C] = 0, 1
        for b in range(B):
            s[b, ::C] = rng.permutation(n) * C
        e = np.minimum(s + rng.integers(0, T // 2, (B, T), dtype=np.int32), T - 1)
    same_best(moc, g, C, R, s, e.astype(np.int32), a)


# copies whose starts or ends lie at the ends of 32 bits: sums of them with the radius stay within int
@pytest.mark.parametrize("n,C,R", [(90, 2, 32), (200, 1, 8), (40, 5, 1)])
def test_copies_at_the_ends_of_the_integers(moc, n, C, R):  # noqa: F811
    rng = np.random.default_rng(n + C + R)
    g = graph(rng, n, 2)
    B, T, lim = 10, n * C, np.iinfo(np.int32)
    s, e = (rng.integers(0, T, (B, T)) for _ in range(2))
    s, e, a = np.minimum(s, e), np.maximum(s, e), np.ones((B, T), np.uint8)
    far = np.array([lim.min, lim.min + R, lim.max - R, lim.max, -(1 << 20), 1 << 20, -R, T - 1 + R])
    s = np.where(rng.random((B, T)) < 0.3, rng.choice(far, (B, T)), s).astype(np.int32)
    e = np.where(rng.random((B, T)) < 0.3, rng.choice(far, (B, T)), e).astype(np.int32)
    same_best(moc, g, C, R, s, e, a)


# copies that one move makes live over most of the domain: more blocks of it than a move of a live copy can change
@pytest.mark.parametrize("n,C,R", [(4000, 2, 2), (900, 3, 32), (4300, 1, 1)])
def test_copies_one_position_outside(moc, n, C, R):  # noqa: F811
    rng = np.random.default_rng(n)
    g = graph(rng, n, 1)
    B, T = 6, n * C
    s, e, a = (np.zeros((B, T), t) for t in (np.int32, np.int32, np.uint8))
    s[:, ::C], a[:, ::C] = np.arange(n) * C, 1
    e[:, ::C] = np.maximum(s[:, ::C], T - 1 - rng.integers(0, 9, (B, n), dtype=np.int32))
    for b in range(B):
        at = np.flatnonzero(rng.random(n) < (0.01, 0.5)[b % 2]) * C
        if b < 4:
            e[b, at] = T - 1 + rng.integers(1, R + 2, at.size)
        if b >= 2:
            s[b, at] = -rng.integers(1, R + 2, at.size)
    same_best(moc, g, C, R, s, e, a)
