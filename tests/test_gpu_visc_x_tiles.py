"""The x line solves whose lines go to the threads as flattened items: every
chunk length, lines that are no whole tiles, one tile and several tiles per
workgroup, against the same solves on a field off the 16-byte alignment (one
element per lane, no registers ahead).  Both do the same arithmetic along x;
the bar is the one of the FP64 path, relative L2 <= 1e-12.  Neighbouring lines
hold unrelated values, so an item of another line is an O(1) error."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bcx", [WALL, PERIODIC])
@pytest.mark.parametrize("dims", [(2, 3, 3), (18, 81, 23), (128, 9, 7), (162, 81, 23), (288, 81, 23), (432, 27, 3),
                                  (512, 27, 3), (576, 81, 5), (768, 27, 3), (1024, 27, 3), (96, 162, 211),
                                  (288, 162, 211), (512, 162, 211)])
def test_x_lines_in_tiles(dims, bcx):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(*dims, bcx, PERIODIC, lx=4.0, ly=4.0, lz=6.5, stretch=1.5)
    plan = F.Plan.from_spec(spec)
    g = torch.Generator(device="cuda").manual_seed(sum(dims))
    q = torch.randn(spec.shape, dtype=torch.float64, device="cuda", generator=g)
    off = torch.empty(q.numel() + 1, dtype=q.dtype, device="cuda")[1:].view(q.shape).copy_(q)
    for comp in range(2):
        plan.viscous_solve(q, comp, 3.0 * spec.dx**2)
        plan.viscous_solve(off, comp, 3.0 * spec.dx**2)
        assert off.data_ptr() % 16 == 8
        assert float((off - q).norm() / q.norm()) <= 1e-12
