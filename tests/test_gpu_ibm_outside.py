"""IB transfer of markers beyond the walls (the support is then the last three
nodes and the operators extrapolate): interpolation and spreading up to 20
cells outside in one, two and three directions against the same operators in
long double.  Bar 1e-11 of the sum of |phi_k u_k|: at r cells the weights'
exponents r^2 round at some 3 r^2 2^-53 (1.3e-13 at 20), over three axes."""
import numpy as np
import pytest

from oracle import WALL
from paper_2103_15187_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LD = np.longdouble
N = 24


def _axis(x, face):
    h = LD(1) / N
    x0 = LD(0) if face else h / 2
    m = min(max(int(np.floor((LD(x) - x0) / h + LD(0.5))), 1), N - 2)
    i = np.array([m - 1, m, m + 1])
    d = x0 + i * h - LD(x)
    n = np.exp(((d / h) ** 2).min() - (d / h) ** 2)
    n = n / n.sum()
    dev = np.array([sum(n[r] * (d[q] - d[r]) for r in range(3)) for q in range(3)])
    var = sum(n[q] * n[r] * (d[q] - d[r]) ** 2 for q in range(3) for r in range(q + 1, 3))
    return i, n, dev * (n * d).sum() / var


def _operators(b, comp):
    """Node indices (z, y, x) and phi of marker b, (27,) each."""
    ax = [_axis(b[c], comp == c) for c in range(3)]
    k, j, i = np.meshgrid(*(a[0] for a in ax[::-1]), indexing="ij")
    n = ax[2][1][:, None, None] * ax[1][1][None, :, None] * ax[0][1][None, None, :]
    g = ax[2][2][:, None, None] + ax[1][2][None, :, None] + ax[0][2][None, None, :]
    return (k.ravel(), j.ravel(), i.ravel()), (n * (1 - g)).ravel()


@pytest.mark.parametrize("comp", [0, 1, 2])
def test_markers_outside(comp):
    from paper_2103_15187_amd import fsei as F
    plan = F.Plan(N, N, N, (WALL, WALL), 1.0 / N, 1.0 / N, np.linspace(0.0, 1.0, N + 1))
    r = W.rng(17 + comp)
    xb = []
    for out in (0.3, 1.0, 2.7, 5.2, 9.6, 13.1, 16.4, 20.0):
        for axes in ((0,), (1,), (2,), (0, 1), (1, 2), (0, 1, 2)):
            for side in (0, 1):
                b = r.uniform(0.1, 0.9, 3)
                for c in axes:
                    b[c] = 1.0 + out / N if side else -out / N
                xb.append(b)
    xb = np.array(xb)
    f = r.standard_normal((N, N, N))
    x = torch.from_numpy(xb).cuda()
    got = plan.ib_interpolate(torch.from_numpy(f).cuda(), comp, x).cpu().numpy()
    assert np.isfinite(got).all()
    for b, u in zip(xb, got):
        at, phi = _operators(b, comp)
        w = phi * f[at]
        assert abs(LD(u) - w.sum()) <= 1e-11 * np.abs(w).sum(), (b, u)
    # spreading, one marker at a time: the same operators over the volumes
    one = torch.ones(1, dtype=torch.float64, device="cuda")
    for b in xb[::7]:
        field = torch.zeros((N, N, N), dtype=torch.float64, device="cuda")
        plan.ib_spread(field, comp, torch.from_numpy(b[None]).cuda(), one, one)
        at, phi = _operators(b, comp)
        kk = at[0]
        h = np.full(N, LD(1) / N)
        if comp == 2:
            h[0] = h[0] / 2
        ref = np.zeros((N, N, N), dtype=LD)
        ref[at] = phi * N * N / h[kk]
        assert np.abs(field.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max(), b
