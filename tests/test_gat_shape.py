"""The lane layout of the fused attention kernels (csrc/gat_shape.h, plain host code), for every
number of heads and head width that the entry points take: a head's lanes hold all its columns,
and for the dot product, whose lanes' parts are summed, each column once."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2101_11552_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "gat_shape.h"
int main() {
  for (int dot = 0; dot < 2; ++dot)
    for (int H = 1; H <= 64; ++H)
      for (int D = 1; D <= (dot ? 64 : 300); ++D) {
        if (dot && (D & (D - 1)) != 0) continue;
        const auto t = tfg::rows::gat_shape(H, D, dot != 0);
        std::printf("%d %d %d %d %d %d\n", dot, H, D, t.vec, t.G, t.lps);
      }
}
"""


def test_lanes_cover_the_columns(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "shape.cpp", str(tmp_path / "shape")
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    lines = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == 64 * (300 + 7)
    for line in lines:
        dot, H, D, vec, G, lps = (int(v) for v in line.split())
        held = [min(g * vec, D - vec) + v for g in range(G) for v in range(vec)]
        assert set(held) == set(range(D)), (dot, H, D)
        assert lps in (4, 8, 16, 32, 64) and lps >= min(H * G, 64), (dot, H, D)
        # lanes that share a score are neighbours within a quad, also where a row of
        # more than 64 lanes goes in passes
        share = (4 if G % 4 == 0 else 2 if G % 2 == 0 else 1) if vec == 4 else 1
        assert H * G <= 64 or 64 % share == 0 and G % share == 0, (dot, H, D)
        if dot:
            assert sorted(held) == list(range(D)), (H, D)
            assert G & (G - 1) == 0, (H, D)  # the sum over aligned groups of lanes
