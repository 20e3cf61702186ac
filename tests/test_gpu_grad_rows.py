"""The general gradient kernel (odd rows, rows off the alignment) at the row
lengths where its columns per thread change, against a plain torch gradient of
the returned pressure (bar 1e-13: two products and two sums per value); and
narrow rows at no more time per cell than 1.35 times that of 243 columns."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [(WALL, PERIODIC), (PERIODIC, WALL)])
@pytest.mark.parametrize("nx", [27, 243, 256, 288, 729, 1024, 1152])
def test_gradient_of_the_pressure(nx, bc):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(nx, 9, 7, *bc, lx=4.0, ly=4.0, lz=6.5, stretch=1.5)
    plan = F.Plan.from_spec(spec)
    g = torch.Generator(device="cuda").manual_seed(nx)
    u, v, w = (torch.randn(spec.shape, dtype=torch.float64, device="cuda", generator=g) for _ in range(3))
    dt = 0.7
    un, vn, wn, p = F.project(u, v, w, plan, dt)
    zc = torch.as_tensor(spec.zc(), device="cuda")
    zm = 0.5 * (zc[1:] + zc[:-1])
    ur, vr, wr = u - dt / spec.dx * (p - p.roll(1, 2)), v - dt / spec.dy * (p - p.roll(1, 1)), w.clone()
    wr[1:] -= dt * (p[1:] - p[:-1]) / (zm[1:] - zm[:-1]).view(-1, 1, 1)
    wr[0] = 0.0
    if bc[0] == WALL:
        ur[:, :, 0] = 0.0
    if bc[1] == WALL:
        vr[:, 0, :] = 0.0
    for a, b in ((un, ur), (vn, vr), (wn, wr)):
        assert float((a - b).abs().max()) <= 1e-13 * float(b.abs().max() + dt * p.abs().max() / min(spec.dx, spec.dy))
