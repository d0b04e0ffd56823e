"""GPU parity of the toggle and cut tables where their kernels can go wrong: edges of the blocks of 8
positions, the rows of 64 and 256, one to five copies per node, workgroups of each size, graphs
whose adjacency lists do not fit LDS, and the largest number of copies the calls take."""
import numpy as np
import pytest

import oracle
from test_gpu_cuts import assert_best, assert_same, schedules, to_dev
from test_gpu_search_steps import random_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moc():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2304_14463_amd import moccasin
    moccasin.lib()
    return moccasin


@pytest.mark.parametrize("n,C,B", [(1, 1, 6), (1, 2, 6), (7, 1, 6), (8, 1, 6), (9, 1, 1500), (4, 2, 6), (31, 2, 900), (32, 2, 1500), (33, 2, 6),
                                   (21, 3, 1500), (64, 4, 900), (13, 5, 1500), (129, 2, 6), (511, 2, 900), (1025, 2, 3), (700, 5, 3),
                                   (63, 1, 1500), (130, 1, 900), (1100, 1, 6)])
def test_toggles(moc, n, C, B):
    rng = np.random.default_rng(7 * n + C)
    g = random_graph(rng, n)
    rows = 6 if n < 500 else 3           # repeated beyond that: batches of every workgroup size
    s, e, a = schedules(rng, g, C, rows, wild=True)
    pick = np.arange(B) % rows
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 100, C)
    got = moc.results_to_numpy(moc.moc_eval_toggles(gh, *to_dev(s[pick], e[pick], a[pick])), moc.TOGGLE_SCORE_DTYPE)
    assert (got == got[pick]).all()
    for b in range(rows):
        assert_same(got[b], oracle.toggles(g, 100, C, s[b], e[b], a[b]), f"n={n} C={C} row {b}")
    gh.free()


@pytest.mark.parametrize("n,C,mode,B", [(4, 2, 0, 6), (32, 2, 1, 1500), (33, 2, 0, 600), (21, 3, 1, 1500), (13, 5, 0, 1500), (129, 2, 1, 600),
                                        (511, 2, 0, 600), (129, 2, 0, 6), (900, 3, 1, 3)])
def test_cuts(moc, n, C, mode, B):
    rng = np.random.default_rng(11 * n + C)
    g = random_graph(rng, n)
    rows = 6 if n < 500 else 3           # repeated beyond that: batches of every workgroup size
    s, e, a = schedules(rng, g, C, rows, wild=True)
    pick = np.arange(B) % rows
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 100, C)
    moves, best = moc.moc_eval_cuts(gh, *to_dev(s[pick], e[pick], a[pick]), want_best=True, keep_inputs=mode == 1)
    moves, best = moc.results_to_numpy(moves, moc.TOGGLE_SCORE_DTYPE), moc.results_to_numpy(best, moc.BEST_MOVE_DTYPE)
    assert (moves == moves[pick]).all() and (best == best[pick]).all()
    for b in range(rows):
        want = oracle.cuts(g, 100, C, s[b], e[b], a[b], with_at_peak=True, mode=mode)
        assert_same(moves[b], want, f"n={n} C={C} row {b}")
        assert_best(best[b], want, f"n={n} C={C} row {b}")
    gh.free()


def test_largest_base(moc):
    """T = 8790, a little below the limit: no adjacency lists in LDS, the deepest table of maxima.
    One orderly base; every 40th toggle and cut against the evaluator."""
    n, C = 4395, 2
    T = n * C
    rng = np.random.default_rng(3)
    g = random_graph(rng, n)
    s, e, a = schedules(rng, g, C, 1, wild=False)
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 100, C)
    dev = to_dev(s, e, a)
    got = moc.results_to_numpy(moc.moc_eval_toggles(gh, *dev), moc.TOGGLE_SCORE_DTYPE)[0]
    pick = np.arange(0, T, 40)
    flips = np.repeat(a, len(pick), 0)
    flips[np.arange(len(pick)), pick] ^= 1
    want = oracle.evaluate(g, 100, C, np.repeat(s, len(pick), 0), np.repeat(e, len(pick), 0), flips)
    for i, name in ((2, "violations"), (0, "peak"), (1, "duration")):
        assert (got[name][pick].astype(np.int64) == want[:, i]).all(), name
    for mode in (0, 1):
        moves, best = moc.moc_eval_cuts(gh, *dev, want_best=True, keep_inputs=mode == 1)
        moves = moc.results_to_numpy(moves, moc.TOGGLE_SCORE_DTYPE)[0]
        bm = moc.results_to_numpy(best, moc.BEST_MOVE_DTYPE)[0]
        ok = np.flatnonzero(moves["violations"] >= 0)
        assert ok.size > 0 and int(bm["violations"]) == moves["violations"][ok].min()
        # one step of the search takes that move, and the edited candidate is worth its score
        ws, we, wa = (x.clone() for x in dev)
        if mode == 0:
            count = moc.moc_search_cuts(gh, ws, we, wa, 1)
        else:
            count, _ = moc.moc_search_two_phase(gh, ws, we, wa, 1, 0)
        if int(count[0]):
            after = oracle.evaluate(g, 100, C, ws.cpu().numpy(), we.cpu().numpy(), wa.cpu().numpy())[0]
            assert (after[2], after[0]) == (int(bm["violations"]), int(bm["peak"]))
    gh.free()


@pytest.mark.parametrize("n,C,B,R", [(5, 2, 3, 2), (64, 2, 1100, 3), (130, 2, 1100, 4), (300, 3, 600, 3), (33, 5, 1100, 2), (600, 2, 520, 2),
                                     (64, 2, 3, 16), (130, 4, 1100, 16)])
def test_neighbours_with_ill_formed_copies(moc, n, C, B, R):
    """Bases in which many active copies are not live (start behind end, outside the domain) and some
    have no live copy at all, on either side of the lines between the workgroup sizes; the rows
    repeat.  Table, best move with it and best move alone."""
    rng = np.random.default_rng(13 * n + C + R)
    g = random_graph(rng, n)
    rows, T = 3, n * C
    s, e, a = schedules(rng, g, C, rows, wild=True)
    flip = rng.random(T) < 0.3                       # row 0: a schedule with some of its intervals turned round
    s[0], e[0] = np.where(flip, e[0] + 1, s[0]), np.where(flip, s[0], e[0])
    s[1], e[1], a[1] = rng.integers(1, T + 3, T), 0, 1   # row 1: no live copy
    pick = np.arange(B) % rows
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 100, C)
    dev = to_dev(s[pick], e[pick], a[pick])
    moves, best = (moc.results_to_numpy(x, d) for x, d in zip(moc.moc_eval_neighbours(gh, *dev, R), (moc.MOVE_SCORE_DTYPE, moc.BEST_MOVE_DTYPE)))
    alone = moc.results_to_numpy(moc.moc_eval_neighbours(gh, *dev, R, want_moves=False)[1], moc.BEST_MOVE_DTYPE)
    assert (alone == best).all()
    for r in range(rows):
        assert (moves[r::rows] == moves[r]).all() and (best[r::rows] == best[r]).all(), r
        scores, bm = oracle.neighbours(g, 100, C, s[r], e[r], a[r], R)
        assert (moves[r]["violations"] == scores[:, 0]).all() and (moves[r]["peak"] == scores[:, 1]).all(), r
        assert (int(best[r]["move"]), int(best[r]["violations"]), int(best[r]["peak"])) == bm, r
    gh.free()
