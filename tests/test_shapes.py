"""The rules by which the host picks a kernel's shape (csrc/moc_shapes.h), over all sizes: a small
program of the rules alone, compiled with g++.  No GPU."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_14463_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "moc_shapes.h"
int main(int argc, char** argv) {
  if (argc == 2 && !strcmp(argv[1], "staged"))
    for (int C = 1; C <= 8; ++C)
      for (int n = 1; n * C <= 19455; ++n) printf("%d %d %d\n", C, n, staged_nodes_per_lane(n, C));
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
    """The kernel with the copies in registers is only taken for graphs whose nodes it covers."""
    C, n, u = shapes("staged").T
    taken = u > 0
    assert (n[taken] <= 512 * u[taken]).all()
    assert (u[taken] * C[taken] <= 16).all() and (C[taken] <= 4).all() and np.isin(u, (0, 1, 2, 4, 8)).all()
    # and it is taken wherever an instantiation covers them
    largest = np.array([0, 8, 8, 4, 4, 0, 0, 0, 0])[C] * 512
    assert (taken == (n <= largest)).all()
