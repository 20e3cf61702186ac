"""The near-singular lines and the zero mode (chunked scans of the row-sum
pivots): boxes so wide that every mode line is near-singular, so the whole z
solve is theirs, against the long-double oracle.  Lengths at the edges of the
chunk sizes, and line counts on both sides of the launch of their own.  FP64
bar 1e-12 (rounding of a few hundred positive-factor steps per line).

The reference is the oracle's solve in long double with the pivots in row-sum
form: the oracle's own Thomas rounds sigma against a_k + c_k, which at the
conditions of these boxes (above 1e10) leaves 1e-11 to 1e-8 in long double."""
import numpy as np
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W
from test_gpu_parity import dev, grid_of, host, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BCS = [(WALL, WALL), (PERIODIC, WALL)]


def _reference(f, g):
    from oracle import fsei_oracle as O
    ld = np.longdouble
    Mx, My = O.transform_matrix(g.nx, g.bcx, ld), O.transform_matrix(g.ny, g.bcy, ld)
    fh = O._apply_along(My, O._apply_along(Mx, f.astype(ld), 2), 1)
    sigma = O.eigenvalues(g.ny, g.dy, g.bcy, ld)[:, None] + O.eigenvalues(g.nx, g.dx, g.bcx, ld)[None, :]
    a, c = O.z_coefficients(g, ld)
    sigma[0, 0] = -1                                   # solved apart below
    q, y, ratio, x = np.ones_like(sigma), np.zeros_like(sigma), [], np.empty_like(fh)
    for k in range(g.nz):
        gk = sigma - a[k] * q
        d = gk - c[k]
        q, y = gk / d, (fh[k] - a[k] * y) / d
        x[k] = y
        ratio.append(c[k] / d)
    for k in range(g.nz - 2, -1, -1):
        x[k] -= ratio[k] * x[k + 1]
    x[:, 0, 0] = O.zero_mode_solve(fh[:, 0, 0], g)[0]
    return O._solve_along(Mx, O._solve_along(My, x, 1), 2).astype(np.float64)


def _spec(nx, ny, nz, bc):
    spec = W.small_spec(nx, ny, nz, *bc, lx=4.0e4, ly=3.0e4, lz=6.5, stretch=2.0)
    dz = np.diff(spec.zc()).min()
    top = 4.0 / spec.dx ** 2 + 4.0 / spec.dy ** 2
    assert top < 4.0 / (dz * dz * 9999.0)            # every line below the threshold
    return spec


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("nz", [2, 3, 31, 33, 128, 129, 257, 384, 385, 512, 513, 768, 769, 1000, 1024, 1025, 2048])
def test_every_line_near_singular(nz, bc):
    from paper_2103_15187_amd import fsei as F
    spec = _spec(12 if nz % 2 else 9, 8, nz, bc)
    f = W.rng(nz).standard_normal(spec.shape)
    ref = _reference(f, grid_of(spec))
    plan = F.Plan.from_spec(spec)
    p = plan.poisson_solve(dev(f))
    torch.cuda.synchronize()
    e = rel(host(p), ref)
    print(nz, bc, e)
    assert e <= 1e-12


@pytest.mark.parametrize("dims", [(128, 64, 20), (64, 64, 300), (64, 64, 600), (64, 32, 1100)])
def test_many_near_singular_lines(dims):
    from paper_2103_15187_amd import fsei as F
    spec = _spec(*dims, (WALL, PERIODIC))
    f = W.rng(7).standard_normal(spec.shape)
    ref = _reference(f, grid_of(spec))
    p = F.Plan.from_spec(spec).poisson_solve(dev(f))
    assert rel(host(p), ref) <= 1e-12
