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


@pytest.mark.parametrize("n,C,B,mode", [(2, 2, 6, 0), (9, 2, 6, 1), (63, 2, 9, 0), (64, 2, 9, 1), (65, 3, 9, 1), (129, 4, 6, 1), (50, 5, 6, 1),
                                        (257, 2, 300, 1), (257, 2, 600, 0), (512, 3, 4, 1), (1100, 2, 3, 0), (2190, 4, 3, 0), (2190, 4, 3, 1),
                                        (2900, 2, 3, 0)])
def test_cuts_follow_the_oracle(moc, n, C, B, mode):
    """The descent by cuts (mode 0) and by cuts that keep the inputs (mode 1): counts, rows and, for
    mode 0, the last step's choice.  Bases with and without violations, batches on either side of
    the lines between the workgroup sizes (the rows repeat beyond the first nine)."""
    import torch
    rng = np.random.default_rng(31 * n + C + mode)
    g = random_graph(rng, n)
    rows, steps = min(B, 9), 12 if n < 300 else 5 if n < 2000 else 1
    s, e, a = schedules(rng, g, C, rows, wild=True)
    budget = int(0.8 * np.median(oracle.evaluate(g, 0, C, s, e, a)[::3, 0]))
    pick = np.arange(B) % rows
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(s[pick], e[pick], a[pick])
    last = torch.full((B, 16), 0x55, dtype=torch.uint8, device="cuda")
    if mode == 1:
        count, merges = moc.moc_search_two_phase(gh, ds, de, da, steps, 0)
        assert (merges.cpu().numpy() == 0).all()
    else:
        count = moc.moc_search_cuts(gh, ds, de, da, steps, work_best=last)
    count, gs, ge, ga = count.cpu().numpy(), ds.cpu().numpy(), de.cpu().numpy(), da.cpu().numpy()
    last = moc.results_to_numpy(last, moc.BEST_MOVE_DTYPE)
    applied = 0
    for r in range(rows):
        k, ws, we, wa = oracle.search_cuts(g, budget, C, s[r], e[r], a[r], steps, mode=mode)
        left = oracle.evaluate(g, budget, C, ws, we, wa)[0]
        after = (int(left[2]), int(left[0]))   # violations, peak
        for b in range(r, B, rows):
            assert count[b] == k, (b, count[b], k)
            assert (ga[b] == wa).all() and (gs[b] == ws).all() and (ge[b] == we).all(), b
            if mode == 0:   # the last step's choice and its score; a step that found nothing leaves none behind
                assert (int(last[b]["move"]) < 0) == (k < steps), b
                assert (int(last[b]["violations"]), int(last[b]["peak"])) == (after if k == steps else (0, 0)), b
        applied += k
    assert applied > 0 or n < 60
    gh.free()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n,C,B,duplicates", [(40, 2, 3, False), (40, 2, 3, True), (150, 2, 600, False), (150, 3, 6, True), (150, 2, 1500, True),
                                              (260, 2, 1500, False), (130, 4, 9, False)])
def test_cuts_with_equal_peaks_and_many_inputs(moc, n, C, B, duplicates, mode):
    """Sizes 1 to 3, so that many positions share the peak and many moves their score, and up to 14
    inputs per node, more than the lanes that score a move; with and without edges listed twice."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(n + C + mode)
    edges = [(int(u), v) for v in range(1, n) for u in rng.integers(max(0, v - 30), v, size=rng.integers(1, 15))]
    g = graph_from_edges(n, sorted(edges if duplicates else set(edges)), rng.integers(1, 4, n), rng.integers(1, 9, n))
    rows, steps = 3, 14
    s, e, a = schedules(rng, g, C, 3 * rows, wild=False)
    s, e, a = s[::3], e[::3], a[::3]   # the orderly ones
    e[2, ::C] = np.maximum(s[2, ::C], e[2, ::C] - rng.integers(0, 2, n) * C)   # some outputs end early: violations
    assert (oracle.evaluate(g, 0, C, s, e, a)[:2, 2] == 0).all()
    budget = int(0.5 * oracle.evaluate(g, 0, C, s, e, a)[0, 0])
    pick = np.arange(B) % rows
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(s[pick], e[pick], a[pick])
    if mode == 1:
        count, merges = moc.moc_search_two_phase(gh, ds, de, da, steps, 0)
    else:
        count = moc.moc_search_cuts(gh, ds, de, da, steps)
    count, gs, ge, ga = count.cpu().numpy(), ds.cpu().numpy(), de.cpu().numpy(), da.cpu().numpy()
    for r in range(rows):
        k, ws, we, wa = oracle.search_cuts(g, budget, C, s[r], e[r], a[r], steps, mode=mode)
        same = (count[r::rows] == k) & (ga[r::rows] == wa).all(1) & (gs[r::rows] == ws).all(1) & (ge[r::rows] == we).all(1)
        assert same.all(), (r, k, np.flatnonzero(~same)[:4])
    assert count.max() > 0
    gh.free()


def moves_through_the_peak(g, C, s, e, a):
    """How many (in-edge, consumer copy) moves have a position at the candidate's peak between the
    start of the producer's copy and the consumer's, and a copy of the producer to spare."""
    _, memory = oracle.profile(g, 0, C, s, e, a)
    before = np.concatenate([[0], np.cumsum(memory == memory.max())])
    live = (a != 0) & (s >= 0) & (s <= e) & (e < g.n * C)
    count = 0
    for v in range(g.n):
        for u in g.in_idx[g.in_ptr[v]:g.in_ptr[v + 1]]:
            copies = np.arange(u * C, u * C + C)
            for k in range(v * C, v * C + C):
                covering = copies[live[copies] & (s[copies] < s[k]) & (e[copies] >= s[k])]
                if live[k] and covering.size and (a[copies] == 0).any():
                    count += int(before[s[k]] > before[s[covering].max() + 1])
    return count


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n,degree,B", [(900, 6, 1), (800, 7, 300), (800, 7, 1024)])
def test_cuts_with_more_moves_than_the_lists_hold(moc, mode, n, degree, B):
    """Chains of long edges across one peak: more moves pass the sieve of a base without violations
    than the longest lists hold (2048), and all of them are scored after all.  Workgroups of 1024, 512
    and 256 threads."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    C = 2
    rng = np.random.default_rng(4)
    half = n // 2
    edges = sorted({(u, half + int(v)) for u in range(half) for v in rng.integers(0, n - half, degree)} | {(u, u + 1) for u in range(half)})
    g = graph_from_edges(n, edges, rng.integers(1, 40, n), rng.integers(1, 9, n))
    s = np.zeros((1, n * C), np.int32); e = s.copy(); a = np.zeros((1, n * C), np.uint8)
    last = np.arange(n) * C
    for u, v in edges:
        last[u] = max(last[u], v * C)
    s[0, ::C], e[0, ::C], a[0, ::C] = np.arange(n) * C, last, 1
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 1000, C)
    ds, de, da = to_dev(*(np.repeat(x, B, 0) for x in (s, e, a)))
    if mode == 1:
        count, _ = moc.moc_search_two_phase(gh, ds, de, da, 3, 0)
    else:
        count = moc.moc_search_cuts(gh, ds, de, da, 3)
    k, ws, we, wa = oracle.search_cuts(g, 1000, C, s[0], e[0], a[0], 3, mode=mode)
    assert (count.cpu().numpy() == k).all() and k == 3
    assert min(moves_through_the_peak(g, C, s[0], e[0], a[0]), moves_through_the_peak(g, C, ws, we, wa)) > 2048
    assert (da.cpu().numpy() == wa).all() and (ds.cpu().numpy() == ws).all() and (de.cpu().numpy() == we).all()
    gh.free()


@pytest.mark.parametrize("C,n,B", [(2, 200, 300), (2, 200, 600), (2, 202, 1024), (3, 150, 300), (3, 150, 1024), (5, 120, 1024), (5, 120, 400)])
def test_cuts_with_more_moves_than_the_groups_take_at_once(moc, C, n, B):
    """Outputs of three sizes held across one peak: hundreds of moves with the same bound, which are scored
    together, in the workgroups of 256 and 512 threads by one lane each."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(n + C)
    half = n // 2
    edges = sorted({(u, half + int(v)) for u in range(half) for v in rng.integers(0, n - half, 4)} | {(u, u + 1) for u in range(half)})
    g = graph_from_edges(n, edges, rng.integers(1, 4, n), rng.integers(1, 9, n))
    s = np.zeros((1, n * C), np.int32); e = s.copy(); a = np.zeros((1, n * C), np.uint8)
    last = np.arange(n) * C
    for u, v in edges:
        last[u] = max(last[u], v * C)
    s[0, ::C], e[0, ::C], a[0, ::C] = np.arange(n) * C, last, 1
    budget, steps = int(oracle.evaluate(g, 0, C, s, e, a)[0, 0]) // 3, 10
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(*(np.repeat(x, B, 0) for x in (s, e, a)))
    count = moc.moc_search_cuts(gh, ds, de, da, steps).cpu().numpy()
    k, ws, we, wa = oracle.search_cuts(g, budget, C, s[0], e[0], a[0], steps)
    assert min(moves_through_the_peak(g, C, s[0], e[0], a[0]), moves_through_the_peak(g, C, ws, we, wa)) > 100 and k > 1
    assert (count == k).all()
    assert (da.cpu().numpy() == wa).all() and (ds.cpu().numpy() == ws).all() and (de.cpu().numpy() == we).all()
    gh.free()


@pytest.mark.parametrize("C,n,B,smaller", [(2, 200, 300, 6), (2, 200, 600, 3), (2, 202, 1024, 5), (2, 260, 1024, 2), (3, 150, 1024, 4), (5, 120, 1024, 3)])
def test_cuts_scored_by_lanes_and_then_by_groups(moc, C, n, B, smaller):
    """Hundreds of moves share the lowest bound and are scored first, one lane each; a few with a higher bound
    follow, a group of lanes each.  The best of both rounds counts, in whichever lane it was found."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(n + C)
    half = n // 2
    edges = sorted({(u, half + int(v)) for u in range(half) for v in rng.integers(0, n - half, 4)} | {(u, u + 1) for u in range(half)})
    size = np.full(n, 3)
    size[rng.choice(half, smaller, replace=False)] = 2
    g = graph_from_edges(n, edges, size, rng.integers(1, 9, n))
    s = np.zeros((1, n * C), np.int32); e = s.copy(); a = np.zeros((1, n * C), np.uint8)
    last = np.arange(n) * C
    for u, v in edges:
        last[u] = max(last[u], v * C)
    s[0, ::C], e[0, ::C], a[0, ::C] = np.arange(n) * C, last, 1
    budget, steps = int(oracle.evaluate(g, 0, C, s, e, a)[0, 0]) // 3, 30
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(*(np.repeat(x, B, 0) for x in (s, e, a)))
    count = moc.moc_search_cuts(gh, ds, de, da, steps).cpu().numpy()
    k, ws, we, wa = oracle.search_cuts(g, budget, C, s[0], e[0], a[0], steps)
    assert k > 1
    assert (count == k).all()
    assert (da.cpu().numpy() == wa).all() and (ds.cpu().numpy() == ws).all() and (de.cpu().numpy() == we).all()
    gh.free()


@pytest.mark.parametrize("call", ["cuts", "two_phase"])
def test_more_candidates_than_a_launch_takes(moc, call):
    """2^21 candidates go into a launch of a descent: a batch that needs a second one, whose
    candidates, counts and choices begin where the first one's end."""
    import torch
    rng = np.random.default_rng(21)
    n, C, B = 8, 2, (1 << 21) + 301
    g = random_graph(rng, n)
    rows = 9
    s, e, a = recomputed(rng, g, C, rows)
    budget = int(0.8 * np.median(oracle.evaluate(g, 0, C, s, e, a)[:, 0]))
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    pick = torch.arange(B, device="cuda") % rows
    ds, de, da = (x[pick].contiguous() for x in to_dev(s, e, a))
    if call == "cuts":
        last = torch.full((B, 16), 0x55, dtype=torch.uint8, device="cuda")
        counts = [moc.moc_search_cuts(gh, ds, de, da, 3, work_best=last)]
        assert (last == last[:rows][pick]).all()
        want = [oracle.search_cuts(g, budget, C, s[r], e[r], a[r], 3) for r in range(rows)]
    else:
        counts = list(moc.moc_search_two_phase(gh, ds, de, da, 3, 3, 8))
        want = [oracle.search_two_phase(g, budget, C, s[r], e[r], a[r], 3, 3, 8) for r in range(rows)]
    assert all(max(w[i] for w in want) > 0 for i in range(len(counts)))
    for got, i in zip((ds, de, da), (-3, -2, -1)):
        assert (got == torch.from_numpy(np.stack([w[i] for w in want])).cuda()[pick]).all(), i
    for i, got in enumerate(counts):
        assert (got == torch.tensor([w[i] for w in want], dtype=torch.int32, device="cuda")[pick]).all(), i
    gh.free()


@pytest.mark.parametrize("n,C,B,R,steps", [(1, 1, 3, 1, 2), (20, 2, 6, 3, 9), (64, 2, 1200, 2, 5), (65, 3, 600, 2, 4), (40, 5, 9, 16, 4),
                                           (300, 4, 3, 4, 3), (700, 2, 520, 2, 2)])
def test_moves_follow_the_oracle(moc, n, C, B, R, steps):
    """The descent by single-field moves: some candidates stop at once, some run out of steps; the
    rows repeat beyond the first nine."""
    rng = np.random.default_rng(17 * n + C + R)
    g = random_graph(rng, n)
    rows = min(B, 9 if n < 100 else 3)
    s, e, a = schedules(rng, g, C, rows, wild=True)
    budget = int(0.9 * oracle.evaluate(g, 0, C, s, e, a)[0, 0])
    pick = np.arange(B) % rows
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, budget, C)
    ds, de, da = to_dev(s[pick], e[pick], a[pick])
    count = moc.moc_search_moves(gh, ds, de, da, R, steps).cpu().numpy()
    gs, ge = ds.cpu().numpy(), de.cpu().numpy()
    assert (da.cpu().numpy() == a[pick]).all()
    for r in range(rows):
        k, ws, we = oracle.search_moves(g, budget, C, s[r], e[r], a[r], R, steps)
        for b in range(r, B, rows):
            assert count[b] == k, (b, count[b], k)
            assert (gs[b] == ws).all() and (ge[b] == we).all(), b
    gh.free()


@pytest.mark.parametrize("duplicates", [False, True])
@pytest.mark.parametrize("C,inputs,B", [(2, 17, 3), (2, 40, 600), (2, 63, 3), (2, 65, 3), (2, 80, 300), (2, 130, 1500), (2, 255, 3), (2, 256, 3), (2, 300, 600),
                                        (2, 520, 3), (3, 64, 3), (3, 100, 600), (5, 90, 3), (5, 270, 600)])
def test_keeping_cuts_with_a_few_of_many_inputs_kept(moc, C, inputs, B, duplicates):
    """Producers with many inputs of which a few are kept: around the number from which a graph has the kernel for
    it and the numbers of inputs that share a bit there."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(inputs + 10 * C + duplicates)
    n = inputs + 90
    edges = {(v - 1, v) for v in range(1, n)}
    wide = [inputs + 5, inputs + 15, inputs + 25]   # the second is gone when the others are needed again
    for u, v in zip(wide, (n - 5, inputs + 50, n - 20)):
        edges |= {(int(w), u) for w in rng.choice(inputs + 3, inputs, replace=False)} | {(u, v)}
    edges |= {(w, n - 1) for w in range(inputs) if w % 9 != 0}   # these inputs are held anyway
    edges = sorted(edges) + ([(int(w), wide[i % 3]) for i, w in enumerate(rng.integers(0, inputs, 40))] if duplicates else [])
    size = rng.integers(1, 4, n)
    size[wide], size[inputs + 40:inputs + 60] = 20 * inputs + rng.integers(2000, 2600, 3), rng.integers(20, 60, 20)
    g = graph_from_edges(n, sorted(edges), size, rng.integers(1, 9, n))
    assert np.diff(g.in_ptr).max() >= inputs
    s = np.zeros((1, n * C), np.int32); e = s.copy(); a = np.zeros((1, n * C), np.uint8)
    last = np.arange(n) * C
    for u, v in edges:
        last[u] = max(last[u], v * C)
    s[0, ::C], e[0, ::C], a[0, ::C] = np.arange(n) * C, last, 1
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 10, C)
    ds, de, da = to_dev(*(np.repeat(x, B, 0) for x in (s, e, a)))
    count, _ = moc.moc_search_two_phase(gh, ds, de, da, 8, 0)
    k, ws, we, wa = oracle.search_cuts(g, 10, C, s[0], e[0], a[0], 8, mode=1)
    assert k > 1 and all(wa[u * C + 1] for u in wide)
    assert (count.cpu().numpy() == k).all()
    assert (da.cpu().numpy() == wa).all() and (ds.cpu().numpy() == ws).all() and (de.cpu().numpy() == we).all()
    gh.free()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("C,n,B,consumers", [(2, 120, 3, 31), (2, 120, 3, 34), (2, 180, 600, 70), (2, 180, 1500, 40), (3, 150, 300, 60), (5, 100, 6, 50)])
def test_cuts_of_producers_with_many_consumers(moc, mode, C, n, B, consumers):
    """Producers read all along the schedule, on either side of the number of consumers from which the sieve of
    the keeping cuts does not walk them."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    rng = np.random.default_rng(n + consumers + C)
    edges = {(v - 1, v) for v in range(1, n)} | {(int(u), v) for v in range(2, n) for u in rng.integers(max(0, v - 25), v, 2)}
    for u in (2, 9, 17, 30):
        edges |= {(u, int(v)) for v in rng.choice(np.arange(u + 1, n), min(consumers, n - u - 1), replace=False)}
    size = rng.integers(1, 30, n)
    size[[2, 9, 17, 30]] = rng.integers(400, 600, 4)
    g = graph_from_edges(n, sorted(edges), size, rng.integers(1, 9, n))
    s = np.zeros((1, n * C), np.int32); e = s.copy(); a = np.zeros((1, n * C), np.uint8)
    last = np.arange(n) * C
    for u, v in edges:
        last[u] = max(last[u], v * C)
    s[0, ::C], e[0, ::C], a[0, ::C] = np.arange(n) * C, last, 1
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 10, C)
    ds, de, da = to_dev(*(np.repeat(x, B, 0) for x in (s, e, a)))
    count = moc.moc_search_two_phase(gh, ds, de, da, 12, 0)[0] if mode == 1 else moc.moc_search_cuts(gh, ds, de, da, 12)
    k, ws, we, wa = oracle.search_cuts(g, 10, C, s[0], e[0], a[0], 12, mode=mode)
    assert k > 0
    assert (count.cpu().numpy() == k).all()
    assert (da.cpu().numpy() == wa).all() and (ds.cpu().numpy() == ws).all() and (de.cpu().numpy() == we).all()
    gh.free()


def wide_producers(rng):
    """Two large outputs, each made from more than 130 small ones that nothing else needs later and
    consumed far behind the peak: a keeping cut of one keeps all of its inputs.  The inputs are listed
    in no order and some of them twice or three times, next to each other and far apart."""
    from paper_2304_14463_amd.inputs import graph_from_edges
    n, u1, u2 = 260, 150, 155
    edges = [(w, u1) for w in range(140)] + [(w, u2) for w in range(10, 150)]
    edges += [(v - 1, v) for v in range(156, n)] + [(v, 259) for v in range(160, 200, 3)]
    edges += [(u1, 156), (u1, 230), (u2, 157), (u2, 236), (3, 225), (70, 228)]
    size = rng.integers(1, 4, n)
    size[[u1, u2]], size[160:200] = (2000, 1700), rng.integers(20, 60, 40)
    g = graph_from_edges(n, edges, size, rng.integers(1, 9, n))
    ptr, idx = list(g.in_ptr), list(g.in_idx)
    for u in (u1, u2):
        listed = idx[ptr[u]:ptr[u + 1]]
        listed = [listed[i] for i in rng.permutation(len(listed))]
        listed = listed[:63] + [listed[62]] * 2 + listed[63:100] + listed[5:9] + listed[100:] + [listed[70], listed[2]]
        more = len(listed) - (ptr[u + 1] - ptr[u])
        idx[ptr[u]:ptr[u + 1]] = listed
        ptr[u + 1:] = [x + more for x in ptr[u + 1:]]
    g.in_ptr, g.in_idx = np.asarray(ptr, np.int32), np.asarray(idx, np.int32)
    assert g.in_ptr[-1] == len(idx)
    return g, (u1, u2)


@pytest.mark.parametrize("C,B", [(2, 1), (2, 300), (2, 600), (2, 1500), (3, 4), (5, 4)])
def test_keeping_cut_of_a_producer_with_many_inputs(moc, C, B):
    """The edit of a keeping cut takes the producer's inputs 64 at a time: three rounds, with inputs
    listed again in the same round and in a later one.  One step keeps over 130 inputs; after it the
    staged profile, maxima and counts have to be those of the edited candidate, or the next steps go
    another way than the oracle's.  Workgroups of each size."""
    g, producers = wide_producers(np.random.default_rng(C))
    n, T = g.n, g.n * C
    s, e, a = np.zeros((1, T), np.int32), np.zeros((1, T), np.int32), np.zeros((1, T), np.uint8)
    pos, last = np.arange(n) * C, np.arange(n) * C
    for v in range(n):
        for u in g.in_idx[g.in_ptr[v]:g.in_ptr[v + 1]]:
            last[u] = max(last[u], pos[v])
    s[0, ::C], e[0, ::C], a[0, ::C] = pos, last, 1
    s, e, a = (np.repeat(x, min(B, 2), 0) for x in (s, e, a))
    if B > 1:                              # the second row: a base with violations (every move scored)
        a[1, 240 * C] = 0
    gh = moc.moc_graph_upload(n, g.in_ptr, g.in_idx, g.size, g.dur, 100, C)
    pick = np.arange(B) % len(s)
    for steps in (1, 6):
        ds, de, da = to_dev(s[pick], e[pick], a[pick])
        count, _ = moc.moc_search_two_phase(gh, ds, de, da, steps, 0)
        count, gs, ge, ga = count.cpu().numpy(), ds.cpu().numpy(), de.cpu().numpy(), da.cpu().numpy()
        for r in range(len(s)):
            k, ws, we, wa = oracle.search_cuts(g, 100, C, s[r], e[r], a[r], steps, mode=1)
            if r == 0:                     # what the test is about did happen
                assert k >= min(steps, 3) and any(wa[u * C + 1] for u in producers) and (we[::C] != e[0, ::C]).sum() > 130
            assert (count[r::len(s)] == k).all()
            for got, want in ((gs, ws), (ge, we), (ga, wa)):
                assert (got[r::len(s)] == want).all(), (steps, r)
    gh.free()
