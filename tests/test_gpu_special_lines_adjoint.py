"""Near-singular lines of the transposed z solve (through T^T = dz T dz^-1) by
themselves: dLoss/dp is one near-singular x mode times a z profile and the
other gradients are 0, so the adjoint's u component is the x difference of the
transposed solve of that line, dx of order 1 here so that nothing cancels.
Against the long-double row-sum solve, bar 1e-12 (some hundred steps of
positive factors per line, two differences)."""
import numpy as np
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W
from test_gpu_parity import dev, grid_of, host, rel
from test_gpu_special_lines import _reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [100, 129, 300, 385, 512, 700, 768, 1000, 1500])
@pytest.mark.parametrize("nx", [27, 32])
def test_transposed_line(nx, nz):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(nx, 8, nz, WALL, PERIODIC, lx=1.0 * nx, ly=1.0, lz=2.0, stretch=1.5)
    g = grid_of(spec)
    zc = spec.zc()
    dz = np.diff(zc)
    lam = 4.0 / spec.dx ** 2 * np.sin(np.pi / (2 * nx)) ** 2
    assert lam < 4.0 / (dz.min() ** 2 * 9999.0)        # mode (1, 0) is near-singular
    x = np.cos(np.pi * (np.arange(nx) + 0.5) / nx)
    q = W.rng(nx + nz).standard_normal((nz, 1, 1)) * np.ones((1, 8, 1)) * x
    z = lambda: torch.zeros(spec.shape, dtype=torch.float64, device="cuda")   # noqa: E731
    gu, gv, gw = z(), z(), z()
    dt = 0.7
    F.Plan.from_spec(spec).project_backward(gu, gv, gw, dev(np.ascontiguousarray(q)), dt=dt)
    s = _reference(q / dz[:, None, None], g) * dz[:, None, None] / dt
    ref = np.zeros_like(s)
    ref[:, :, 1:] = (s[:, :, :-1] - s[:, :, 1:]) / spec.dx
    e = rel(host(gu), ref)
    print(nx, nz, e)
    assert e <= 1e-12
