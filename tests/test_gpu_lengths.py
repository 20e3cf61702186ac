"""Every transform length with kernels of its own, as the x and as the y
direction, against the FP64 oracle in every precision mode and the adjoint
(bars as for the longest lines: FP64 at 1e-12 or three times the oracle's own
error against long double, plain FP32 at 2e-4, where a mistake in a radix, a
tile edge or a ragged row gives O(1) errors).  x lines: 18 rows per plane, not a multiple of
any row tile; y lines: 27 and 36 columns, unpaired and ragged column tiles."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W
from paper_2103_15187_amd._build import LENGTHS
from test_gpu_parity import _check_all_precisions

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("axis", ["x", "y"])
def test_every_compiled_length(n, axis):
    odd = LENGTHS.index(n) % 2
    bc = (WALL, PERIODIC) if odd else (PERIODIC, WALL)
    if axis == "x":
        dims = (n, 18, 3)
    else:
        dims, bc = ((27 if odd else 36), n, 3), bc[::-1]
    for b in (bc, bc[::-1]):
        spec = W.small_spec(*dims, *b, lx=4.0, ly=4.0, lz=6.5, stretch=1.5)
        _check_all_precisions(spec, n, bar32=2e-4)


@pytest.mark.parametrize("dims,bc", [((96, 16, 5), (WALL, PERIODIC)), ((768, 6, 3), (PERIODIC, WALL))])
def test_fields_off_the_pair_alignment(dims, bc):
    """8-byte aligned fields take the kernels with the length from the arguments."""
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(*dims, *bc, lx=4.0, ly=4.0, lz=6.5, stretch=1.5)
    plan = F.Plan.from_spec(spec)
    g = torch.Generator(device="cuda").manual_seed(5)
    q = [torch.randn(spec.shape, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    off = [torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t) for t in q]
    p = plan.project(*q, dt=0.7)
    po = plan.project(*off, dt=0.7)
    for a, b in zip([*off, po], [*q, p]):
        assert float((a - b).norm() / b.norm()) <= 1e-12
