"""Rows that the fused x inverse + gradient reads (xg_in_row of fsei_plan.h, the
kernel's own addressing), compiled for the host: every line of every tile lies
in its plane, the lines that count are the halo row and the eight own rows in
order, and the last sequence's zero line addresses one of the tile's rows."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_15187_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "fsei_plan.h"
using namespace fsei;
int main() {
    for (int ny = kXgRows; ny <= 1024; ny += kXgRows)
        for (int j0 = 0; j0 < ny; j0 += kXgRows)
            for (int l = 0; l < 2 * kXgSeq; ++l) {
                const int row = xg_in_row(l / 2, l % 2, j0, ny);
                const bool zero = l > kXgRows;   // after the halo row and the own rows
                const int want = l == 0 ? (j0 + ny - 1) % ny : j0 + l - 1;
                if (row < 0 || row >= ny || (zero ? row / kXgRows != j0 / kXgRows : row != want)) {
                    std::printf("ny %d j0 %d line %d: row %d\n", ny, j0, l, row);
                    return 1;
                }
            }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_input_row_lies_in_the_plane(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
