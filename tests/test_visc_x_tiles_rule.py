"""Tiles per workgroup of the viscous x solves (visc_x_tiles of fsei_plan.h),
compiled for the host: the tile steps of all rounds of the CUs, with 2.5 more
per workgroup for its tables and first tile, are at most those of one and of
four tiles per workgroup, whatever the length and the number of lines."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_15187_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "fsei_plan.h"
using namespace fsei;
// tile steps of all rounds: at most `per_cu` workgroups of t tiles of 8 lines on a CU
double steps(long nlines, int t, long per_cu) {
    const long groups = (nlines + 8 * t - 1) / (8 * t), slots = 256 * per_cu;
    return (double)((groups + slots - 1) / slots) * (t + 2.5);
}
int main() {
    // rows, workgroups per CU (LDS 160 KB; tables and tile of one: see the kernel)
    const int cases[][2] = {{128, 7}, {384, 3}, {512, 2}, {768, 1}, {1024, 1}};
    for (auto& c : cases)
        for (long nlines = 4; nlines < 400000; nlines += 1 + nlines / 7) {
            const int t = visc_x_tiles(nlines, c[0], visc_chunk(c[0]), 256);
            if (t < 1 || t > 4) return std::printf("n %d lines %ld: %d tiles\n", c[0], nlines, t), 1;
            const double s = steps(nlines, t, c[1]), s1 = steps(nlines, 1, c[1]), s4 = steps(nlines, 4, c[1]);
            if (s > s1 || s > s4)
                return std::printf("n %d lines %ld: %d tiles, %g steps (1: %g, 4: %g)\n", c[0], nlines, t, s, s1, s4), 1;
        }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_never_more_steps_than_one_or_four_tiles(tmp_path):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
