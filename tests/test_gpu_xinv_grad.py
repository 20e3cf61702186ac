"""The fused x inverse + gradient (even lengths from 256 to 768, whole 8-row
tiles, grids of at least 32 planes of one tile per CU) against the two separate
passes, which fields off the 16-byte alignment take: the same stencils on the
same transforms, so the difference is rounding (relative L2 <= 1e-12, the bar
of the FP64 path).  Forward with and without a pressure output, and the
adjoint; plane chunks with a ragged last one."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _off(t):
    return torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t)


@pytest.mark.parametrize("dims,bc", [((256, 256, 261), (WALL, PERIODIC)), ((288, 64, 1030), (PERIODIC, WALL)),
                                     ((432, 256, 258), (WALL, WALL)), ((512, 512, 131), (PERIODIC, PERIODIC)),
                                     ((576, 256, 257), (WALL, PERIODIC)), ((768, 256, 260), (PERIODIC, WALL))])
def test_fused_against_separate_passes(dims, bc):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(*dims, *bc, lx=4.0, ly=4.0, lz=6.5, stretch=2.0)
    plan = F.Plan.from_spec(spec)
    assert dims[1] // 8 * dims[2] >= 32 * torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device="cuda").manual_seed(sum(dims))
    q = [torch.randn(spec.shape, dtype=torch.float64, device="cuda", generator=g) for _ in range(3)]
    a, b, c = [t.clone() for t in q], [_off(t) for t in q], [t.clone() for t in q]
    plan.set_timing(True)
    pa = plan.project(*a, dt=0.7)
    assert "xinv_grad" in plan.kernel_times()
    plan.reset_timing()
    pb = plan.project(*b, dt=0.7)
    assert "xinv_grad" not in plan.kernel_times()
    plan.set_timing(False)
    plan.project(*c, dt=0.7, want_p=False)
    for x, y in zip([*a, pa], [*b, pb]):
        assert float((x - y).norm() / y.norm()) <= 1e-12
    assert all(torch.equal(x, y) for x, y in zip(a, c))
    a, b = [t.clone() for t in q], [_off(t) for t in q]
    plan.project_backward(*a, None, dt=0.7)
    plan.project_backward(*b, None, dt=0.7)
    for x, y in zip(a, b):
        assert float((x - y).norm() / y.norm()) <= 1e-12
