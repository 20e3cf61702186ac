"""The register bound of the compiled y kernels (y_len_waves of fsei_plan.h), compiled
for the host: the waves per SIMD it asks for are waves that the kernels' LDS
lets a CU hold, at every length, precision and direction."""
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
    const int lengths[] = {
#define LEN(n) n,
        FSEI_LENGTHS(LEN)
    };
    int bad = 0;
    for (int n : lengths)
        for (int elem : {4, 8})
            for (bool inverse : {false, true}) {
                // tile arrays of 64- or 128-byte rows with their pads, twiddles of 2 or 4 tables
                const int pairs = (n <= 512 ? 64 : 32) / elem, pad = (elem == 4 && !inverse) ? 6 : 4;
                const int lds = (2 * pairs * (n + (n >> pad) + 1) + (elem == 4 && !inverse ? 4 : 2) * n) * elem;
                const int fit = 160 * 1024 / lds;
                if (y_len_waves(n, elem, inverse) * 256 > fit * y_len_threads(n, elem) + 255) {
                    std::printf("n %d elem %d inverse %d: %d workgroups fit\n", n, elem, inverse, fit);
                    bad = 1;
                }
            }
    return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_bound_is_attainable(tmp_path):
    src, exe = tmp_path / "y.cpp", tmp_path / "y"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
