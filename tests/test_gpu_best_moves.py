"""The best single-field move without the table of scores, where its kernel does not score every move: the move the
kernel of the table picks among all of them, and the descent as repeated calls of it."""
import numpy as np
import pytest

from test_gpu_neighbours import gpu_neighbours, moc, random_candidates, to_dev  # noqa: F401  (moc: fixture)

pytestmark = pytest.mark.gpu


def graph(rng, n, per_node, size_hi=50, repeat=False):
    from paper_2304_14463_amd.inputs import graph_from_edges
    edges = [(int(u), v) for v in range(1, n) for u in rng.integers(0, v, size=rng.integers(0, 2 * per_node + 1))]
    return graph_from_edges(n, sorted(edges) if repeat else sorted(set(edges)), rng.integers(0, size_hi, n), rng.integers(1, 9, n))


def schedules(rng, g, C, B, R):
    """Rows of every kind: a plain schedule, its perturbations, anything at all."""
    T = g.n * C
    s, e, a = random_candidates(rng, B, T, T, wild=True)
    last = np.full(g.n, 0)
    for v in range(g.n):
        for u in g.in_idx[g.in_ptr[v]:g.in_ptr[v + 1]]:
            last[u] = v
    for b in range(B // 2 + 1):
        s[b], e[b], a[b] = 0, 0, 0
        s[b, ::C] = np.arange(g.n) * C
        e[b, ::C] = np.maximum(last * C, s[b, ::C])
        a[b, ::C] = 1
        if b:
            moves = rng.random((2, T)) < (0.02, 0.3)[b % 2]
            s[b] += np.where(moves[0], rng.integers(-R, R + 1, T), 0).astype(np.int32)
            e[b] += np.where(moves[1], rng.integers(-R, R + 1, T), 0).astype(np.int32)
    return s, e, a


# either side of the sizes at which more threads are taken (T = 256, 1024, 2048, 5000; few and many bases), of the
# sixteen displacements and edges that are looked at together, of the copies a thread asks for ahead
@pytest.mark.parametrize("n,C,R,B,per_node", [
    (128, 2, 1, 6, 2), (129, 2, 8, 6, 2), (512, 2, 9, 6, 2), (513, 2, 16, 6, 2), (1024, 2, 17, 6, 2), (683, 3, 2, 6, 2), (1030, 2, 32, 4, 1),
    (513, 4, 7, 700, 1), (1251, 4, 3, 260, 1), (1025, 1, 31, 600, 2), (60, 5, 15, 900, 8), (60, 2, 8, 900, 25), (300, 3, 4, 40, 12)])
def test_best_move_is_the_table_s(moc, n, C, R, B, per_node):  # noqa: F811
    rng = np.random.default_rng(n * 100 + C * 10 + R)
    g = graph(rng, n, per_node, size_hi=3 if n % 2 else 50, repeat=n == 60)
    s, e, a = schedules(rng, g, C, B, R)
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, int(g.size.sum()) // 3, C)
    _, want = gpu_neighbours(moc, gh, s, e, a, R)
    _, got = gpu_neighbours(moc, gh, s, e, a, R, moves=False)
    bad = [b for b in range(B) if got[b].tobytes() != want[b].tobytes()]
    assert not bad, (bad[:5], got[bad[0]], want[bad[0]])
    gh.free()


@pytest.mark.parametrize("kind", ["many edges", "no edges", "all alike", "nothing active", "no memory"])
def test_best_move_of_unusual_bases(moc, kind):  # noqa: F811
    """More edges than a count of mendable violations can take (32703: it stops); none; bases in which every field
    has the same bound, more of them than wait at once; none to score; no position below the peak."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(len(kind))
    n, C, R = (260, 1, 1) if kind == "many edges" else (400, 2, 8)
    if kind == "many edges":
        edges = [(u, v) for v in range(n) for u in range(v)] + [(0, n - 1)] * 40000
    else:
        edges = [] if kind in ("no edges", "all alike") else [(v - 1, v) for v in range(1, n)]
    g = graph_from_edges(n, edges, np.zeros(n, int) if kind == "no memory" else np.ones(n, int) if kind == "all alike" else rng.integers(1, 9, n),
                         np.ones(n, int))
    s, e, a = schedules(rng, g, C, 6, R)
    T = n * C
    if kind == "many edges":
        s[1], e[1], a[1] = T - 1 - np.arange(T), T - 1, 1      # every edge uncovered
        e[2] = s[2]
    if kind == "all alike":
        s[:], e[:], a[:] = np.arange(T), np.arange(T), 1
        s[1], e[1] = 5, 5                                       # all starts shared
        s[2], e[2] = 0, T - 1
    if kind == "nothing active":
        a[:3] = 0
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 10, C)
    _, want = gpu_neighbours(moc, gh, s, e, a, R)
    _, got = gpu_neighbours(moc, gh, s, e, a, R, moves=False)
    assert got.tobytes() == want.tobytes(), (got, want)
    gh.free()


@pytest.mark.parametrize("n,C,R,B,steps", [(40, 2, 8, 700, 12), (513, 2, 4, 30, 9), (700, 3, 17, 300, 5), (1100, 2, 3, 6, 6)])
def test_descent_is_repeated_best_moves(moc, n, C, R, B, steps):  # noqa: F811
    """One launch for all steps against one call a step: the best move of the table, applied on the host if it lowers
    (violations, max(peak, M), peak)."""
    rng = np.random.default_rng(n + R)
    g = graph(rng, n, 2)
    budget = int(g.size.sum()) // 4
    s, e, a = schedules(rng, g, C, B, R)
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(s, e, a)
    got = moc.moc_search_moves(gh, ds, de, da, R, steps).cpu().numpy()
    ws, we, want = s.copy(), e.copy(), np.zeros(B, int)
    going = np.ones(B, bool)
    for _ in range(steps):
        res = moc.results_to_numpy(moc.moc_eval_batch(gh, *to_dev(ws, we, a)))
        _, best = gpu_neighbours(moc, gh, ws, we, a, R)
        for b in np.flatnonzero(going):
            v, p, q = int(best[b]["violations"]), int(best[b]["peak"]), int(best[b]["move"])
            now = (int(res[b]["violations"]), max(int(res[b]["peak"]), budget), int(res[b]["peak"]))
            if q < 0 or (v, max(p, budget), p) >= now:
                going[b] = False
                continue
            d, field, k = q % (2 * R), (q // (2 * R)) & 1, q // (4 * R)
            (ws, we)[field][b, k] += d - R if d < R else d - R + 1
            want[b] += 1
    assert (got == want).all() and want.max() == steps
    assert (ds.cpu().numpy() == ws).all() and (de.cpu().numpy() == we).all() and (da.cpu().numpy() == a).all()
    gh.free()
