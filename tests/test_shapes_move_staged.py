"""Layouts of the best-move and the staged kernels (csrc/moc_shapes.h) over all sizes the calls take.  No GPU."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_14463_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "moc_shapes.h"
constexpr int kMaxLds = 160 * 1024;
int main(int argc, char**) {
  if (argc == 1)
    for (int T = 1; neighbours_fit(T, kMaxLds); ++T)
      for (int64_t B : {1, 256, 257, 513, 100000}) {
        const int nt = best_threads(T, B, 256, kMaxLds);
        const BmLayout l = bm_layout(T, nt);
        const bool apart = l.base.table >= T && l.base.pre >= l.base.table + l.base.blocks && l.base.packed > l.base.suf + l.base.blocks &&
                           l.base.occ1 >= l.base.packed + T && l.counts >= l.base.scratch + kScratchWords && l.counts % 4 == 0 && l.queue >= l.red + T;
        printf("%d %d %d %d\n", nt, T, l.bytes, apart && l.cap / 2 * 2 >= nt);
      }
  else
    for (int C = 1; C <= 4; ++C)
      for (int n = 1; n <= 8192; ++n)
        for (int64_t B : {1, 769}) {
          const StagedShape s = staged_shape(n, C, B, 256);
          if (s.nodes == 0) continue;
          const int nt = s.nt, T = n * C;
          const SfLayout l = sf_layout(n, C, nt);
          const bool apart = l.cur_off >= T + C && l.bucket_off >= l.cur_off + n && 2 * (l.delta_off - l.bucket_off) >= T &&
                             nt * l.chunk > T && l.chunk % 2 == 1 && l.red_off >= l.delta_off + nt * l.chunk && l.red_off % 4 == 0;
          printf("%d %d %d %d %d\n", nt, (n + nt - 1) / nt, s.nodes, l.bytes, apart);
        }
  return 0;
}
"""


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    at = tmp_path_factory.mktemp("shapes")
    (at / "shapes.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(at / "shapes"), str(at / "shapes.cpp")], check=True)
    return lambda *args: np.array([x.split() for x in subprocess.run([str(at / "shapes"), *args], check=True, capture_output=True,
                                                                     text=True).stdout.splitlines()], dtype=np.int64)


def test_best_move_layout_fits_wherever_the_table_s_does(rows):
    nt, T, size, ok = rows().T
    assert T.max() > 8000 and ok.all() and (size <= 160 * 1024).all()
    assert np.isin(nt, (256, 512, 1024)).all() and (T[nt == 256] <= 1024).all()   # 256 threads ask for all copies ahead


def test_staged_layout_fits_and_covers_every_node(rows):
    nt, per_lane, nodes, size, ok = rows("staged").T
    assert ok.all() and (size <= 160 * 1024).all()
    assert (per_lane <= nodes).all() and (nt[nodes == 4] == 1024).all()
