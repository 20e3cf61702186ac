"""Registers of the general gradient kernel in the built library: rows of up to 256
columns, one per thread, keep all eight waves per SIMD."""
import os
import re

import pytest

from paper_2103_15187_amd import fsei
from test_z_registers import _kernels

pytestmark = pytest.mark.skipif(not os.path.exists(fsei.LIB_PATH), reason="libfsei.so not built")


def test_short_rows_keep_eight_waves():
    regs = {m.group(1): k[".vgpr_count"] for name, k in _kernels().items()
            if (m := re.match(r"_ZN4fsei3dev6k_gradI([fd])[fd]Li2E", name))}
    assert set(regs) == {"f", "d"}
    assert all((n + 7) // 8 * 8 <= 64 for n in regs.values()), regs
