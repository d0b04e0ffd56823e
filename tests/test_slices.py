"""The consumers of every node as the decode kernel walks them (csrc/moc_slices.h): a small program of the
header alone, compiled with g++.  No GPU."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_14463_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "moc_slices.h"
int main(int argc, char** argv) {   // n C m, then m edges (u, v) in the order of u
  int n, C, m;
  if (scanf("%d %d %d", &n, &C, &m) != 3) return 1;
  std::vector<int32_t> ptr(n + 1), idx(m);
  for (int q = 0; q < m; ++q) {
    int u, v;
    if (scanf("%d %d", &u, &v) != 2) return 1;
    ++ptr[u + 1];
    idx[q] = v;
  }
  for (int v = 0; v < n; ++v) ptr[v + 1] += ptr[v];
  if (argc == 3) {   // limit WAVES
    printf("%d\n", slice_degree(n, atoi(argv[2]), ptr.data()));
    return 0;
  }
  std::vector<uint32_t> list = out_slices(n, C, ptr.data(), idx.data());
  if (argc == 2) {   // reads: words the kernel is given; where a wave's rows begin that it reads ahead, 16 waves
    list = slices_for_kernel(n, C, 16, ptr.data(), idx.data());
    printf("%zu\n", list.size());
    for (uint32_t wave = 0; wave < 16; ++wave)
      for (int r = kHeldRows; r < 2 * kHeldRows; ++r) {
        const bool any = wave < list[0];
        const uint32_t at = any ? list[2 + wave] : 0;
        printf("%u\n", row_ahead(any ? at + kSliceLanes : 0, any ? (int)((list[3 + wave] - at) / kSliceLanes) - 1 : -1, r));
      }
    return 0;
  }
  for (uint32_t w : list) printf("%u\n", w);
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    at = tmp_path_factory.mktemp("slices")
    (at / "slices.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(at / "slices"), str(at / "slices.cpp")], check=True)

    def run(n, C, edges, *args):
        text = f"{n} {C} {len(edges)}\n" + "\n".join(f"{u} {v}" for u, v in edges)
        out = subprocess.run([str(at / "slices"), *map(str, args)], input=text, check=True, capture_output=True, text=True).stdout
        return np.array(out.split(), dtype=np.int64)
    return run


@pytest.mark.parametrize("n,C,degree", [(1, 1, 0), (63, 1, 3), (64, 2, 5), (65, 3, 33), (200, 4, 32), (700, 2, 90), (8190, 2, 2)])
def test_every_edge_once(program, n, C, degree):
    """Every node stands in one slice or apart, with its own consumers and no others; lanes and halves that
    hold none lead to node n; nodes apart are those with more than 32."""
    rng = np.random.default_rng(n * 8 + C)
    out = [np.sort(rng.integers(0, n, rng.integers(0, degree + 1))) for _ in range(n)]
    if n > 64:
        out[5] = rng.integers(0, n, 300)   # a hub, with some consumers twice
    edges = [(u, int(v)) for u in range(n) for v in out[u]]
    w = program(n, C, edges)
    stride = 2 * (4 if C == 3 else C)
    slices, apart = int(w[0]), int(w[1])
    begin = w[2:3 + slices]
    aside = w[3 + slices:3 + slices + apart]
    assert begin[0] == 3 + slices + apart and begin[-1] == w.size
    assert sorted(aside) == [u for u in range(n) if len(out[u]) > 32]
    seen, lengths = list(aside), []
    for i in range(slices):
        rows = w[begin[i]:begin[i + 1]].reshape(-1, 64)
        lengths.append(rows.shape[0])
        for lane in range(64):
            node, words = int(rows[0, lane]), rows[1:, lane]
            uses = np.stack([words & 0xFFFF, words >> 16], 1).reshape(-1)
            assert (uses % stride == 0).all()
            uses = uses // stride
            if node == n:
                assert (uses == n).all()
                continue
            seen.append(node)
            k = len(out[node])
            assert list(uses[:k]) == [int(v) for v in out[node]] and (uses[k:] == n).all()
    assert sorted(seen) == list(range(n))
    assert lengths == sorted(lengths, reverse=True)   # the long ones first


@pytest.mark.parametrize("n,C,edges", [
    *[(n, 2, []) for n in (1, 2, 63, 64)], (65, 1, []), (64, 4, []),          # nodes without consumers only
    (1, 2, [(0, 0)] * 33), (3, 1, [(0, 1)] * 33 + [(1, 2)] * 40 + [(2, 0)] * 50),   # every node apart
    (40, 2, [(0, v) for v in range(1, 40)]), (60, 3, [(0, v) for v in range(1, 60)]),   # one apart, the others last
    (128, 4, [(u, u + 64) for u in range(64)]), (128, 2, [(u, u + 64) for u in range(64)] * 5),
    (360, 2, [(u, 300 + (u + k) % 60) for u in range(300) for k in range(33)]),
    (1016, 2, [(u, 956 + (u + k) % 60) for u in range(956) for k in range(33)]),
    (200, 2, [(u, u + 1) for u in range(199)])])
def test_rows_read_ahead_lie_in_the_list(program, n, C, edges):
    """The rows a wave reads whether or not its first slice has them: no word beyond the list, whatever
    slices there are."""
    words, *ahead = program(n, C, sorted(edges), "reads")
    assert len(ahead) == 32 and min(ahead) >= 0 and max(ahead) + 64 <= words


def test_many_consumers_are_listed_apart_where_few_nodes_have_them(program):
    """Apart are the nodes that would keep the other lanes of a slice and the other waves waiting, not all nodes
    of a graph whose nodes have many consumers."""
    def limit(degrees, waves):
        return int(program(len(degrees), 2, [(u, (u + 1 + k) % len(degrees)) for u, d in enumerate(degrees) for k in range(d)], "limit", waves)[0])
    assert limit([3] * 500, 8) == 32 and limit([32] * 500, 8) == 32
    assert limit([40] * 1000, 4) >= 40 and limit([100] * 1000, 4) >= 100 and limit([5, 100] * 500, 4) >= 100
    assert limit([3] * 980 + [200] * 20, 4) < 200 and limit([3] * 1960 + [1000] * 40, 8) < 1000
    assert limit([60] * 1960 + [1000] * 40, 8) in range(60, 1000)   # both
    assert limit([33], 1) == 32 and limit([0], 1) == 32


def test_sizes_beyond_16_bits_have_none(program):
    assert program(19455, 1, []).size > 0
    assert program(8191, 4, []).size > 0 and program(8192, 4, []).size == 0
    assert program(100, 5, []).size == 0
