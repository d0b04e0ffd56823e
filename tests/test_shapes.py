"""The rules by which the host picks a kernel's shape (csrc/moc_shapes.h), over all sizes: a small
program of the rules alone, compiled with g++.  No GPU."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_14463_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "moc_shapes.h"
constexpr int kMaxLds = 160 * 1024;
int main(int argc, char** argv) {
  if (argc == 2 && !strcmp(argv[1], "staged"))
    for (int C = 1; C <= 8; ++C)
      for (int n = 1; n * C <= 19455; ++n)
        for (int64_t B : {1, 256, 768, 769, 100000}) {
          const StagedShape s = staged_shape(n, C, B, 256);
          printf("%d %d %d %d %d\n", C, n, (int)B, s.nt, s.nodes);
        }
  if (argc == 2 && !strcmp(argv[1], "decode"))
    for (int C = 1; C <= 8; ++C)
      for (int n = 1; n * C <= 19455; ++n) {
        const DecodeShape s = decode_shape(n, C);
        const int rounds = s.loop ? 2 : 1;   // the kernel's
        const bool covered = C <= 4 && s.lay.bytes <= kMaxLds && s.lay.T_pad <= 8 * s.nt * rounds && (s.loop || n <= node_slots(C) * s.nt);
        const int any = dc_layout(n, C).bytes;
        const DecodeShape few = decode_shape(n, C, 256, 256);   // a small batch
        const bool as_well = few.loop == s.loop && few.nt >= s.nt && few.nt <= 1024 && (few.nt >= n || few.nt == 1024) && (C > 4 || few.lay.bytes <= kMaxLds);
        printf("%d %d %d %d %d %d %d\n", C, n, decode_fits(n, C, kMaxLds), covered, s.nt, any, as_well);
      }
  if (argc == 5 && !strcmp(argv[1], "descend")) {   // C, edges per node, candidates
    const int C = atoi(argv[2]);
    const int64_t B = atoll(argv[4]);
    for (int n = 1; moves_fit(n * C, kMaxLds); ++n) {
      const int T = n * C, m = (int)(atof(argv[3]) * n);
      const DescendShape s = descend_shape(T, n, m, B, 256, kMaxLds);
      const MvLayout least = mv_layout(T, n, m, descend_words(s.nt) + sift_words(n, 512), true, kMaxLds);
      printf("%d %d %d %d %d %d\n", n, s.nt, s.cap, s.lay.bytes, s.lay.lists != 0, least.lists != 0);
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    """Runs the program with the given arguments; its rows of numbers as an array."""
    at = tmp_path_factory.mktemp("shapes")
    (at / "shapes.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(at / "shapes"), str(at / "shapes.cpp")], check=True)

    def run(*args):
        out = subprocess.run([str(at / "shapes"), *map(str, args)], check=True, capture_output=True, text=True).stdout
        return np.array([line.split() for line in out.splitlines()], dtype=np.int64)
    return run


def test_staged_kernel_holds_every_node(shapes):
    """The kernel with the copies in registers is only taken for graphs whose nodes it covers, in a shape that it is built for."""
    C, n, B, nt, nodes = shapes("staged").T
    taken = nodes > 0
    assert (n[taken] <= (nt * nodes)[taken]).all() and (nt[~taken] == 512).all()
    assert (C[taken] <= 4).all() and np.isin(nodes, (0, 1, 2, 4)).all() and np.isin(nt, (64, 128, 256, 512, 1024)).all()
    assert (nodes[nt == 1024] != 1).all() and (nt[nodes == 4] == 1024).all() and (C[nodes == 4] <= 2).all()
    # and it is taken wherever an instantiation covers them
    largest = np.array([0, 4096, 4096, 2048, 2048, 0, 0, 0, 0])[C]
    assert (taken == (n <= largest)).all()
    # a lane has one node more rarely than a wave is idle, unless the batch is small
    assert ((nodes[B > 768] != 1) | (n[B > 768] <= 64)).all()


@pytest.mark.parametrize("C", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("edges,B", [(3, 1), (3, 32), (3, 300), (2.25, 600), (3, 1024), (6, 1024), (0, 100000)])
def test_descent_keeps_the_adjacency_lists(shapes, C, edges, B):
    """The sieve's lists push the graph's adjacency lists out of LDS only where they would have to be
    shorter than 512, workgroups of fewer than 1024 threads always have the adjacency lists (they are
    not built without), and every size the call takes fits."""
    n, nt, cap, bytes_, lists, lists_with_512 = shapes("descend", C, edges, B).T
    assert n.size * C > 8700
    assert (bytes_ <= 160 * 1024).all()
    assert (lists[nt < 1024] == 1).all() and np.isin(nt, (256, 512, 1024)).all()
    assert np.isin(cap, (256, 512, 1024, 2048)).all()
    lost = n[lists < lists_with_512]
    assert lost.size == 0, f"n = {lost.min()} .. {lost.max()}"


def test_decode_kernels_hold_every_size_the_call_takes(shapes):
    """C <= 4: the kernel with one lane per node at every size, with as few threads as hold the candidate;
    more copies: the one for any C.  The largest sizes are those of the call's first kernels."""
    C, n, fits, covered, nt, any_bytes, few_as_well = shapes("decode").T
    fits, few = fits == 1, C <= 4
    assert (covered[fits & few] == 1).all(), n[fits & few & (covered == 0)]
    assert (few_as_well[fits & few] == 1).all()
    assert (any_bytes[fits & ~few] <= 160 * 1024).all()
    assert [int(n[fits & (C == c)].max()) for c in range(1, 9)] == [16367, 8183, 5115, 4091, 3273, 2727, 2338, 2045]
    for c, per_lane in ((1, 4), (2, 4), (3, 2), (4, 2)):
        at = C == c
        least = np.ceil(np.maximum(n[at] / per_lane, (c * n[at] + 2) / 8))
        assert (nt[at] == np.clip(2 ** np.ceil(np.log2(np.maximum(least, 64))), 64, 1024)).all()
