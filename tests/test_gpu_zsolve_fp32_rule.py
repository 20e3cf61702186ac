"""FP32 z solves on the other side of each line of the tiling's rule (bars and
checks of test_gpu_zsolve_fp32.py): nx / 2 odd with many tiles (the 1024-thread
form) at 13 to 32 chunks of 4 and at 8 rows per chunk, few chunks beside them,
and more than 20 tiles per CU of 16 rows per chunk."""
import pytest

import test_gpu_zsolve_fp32 as base
from oracle import PERIODIC, WALL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(162, 96, 48), (162, 96, 49), (162, 96, 128), (54, 162, 129), (54, 162, 256),
                                      (512, 324, 385)])
def test_other_side_of_the_rule(nx, ny, nz):
    base.test_fp32_z_lines(nx, ny, nz, (WALL, PERIODIC))
