"""The FP32 z solve of up to 512 rows on even widths: every chunk length at its
first and last line length, widths that are whole tiles of 32 modes, ragged
and below one tile, against the FP64 plan of the same grid (relative L2 <=
2e-4, the bar of plain FP32 on other shapes: rounding is 1e-6, a mistake at a
tile edge or a chunk boundary O(1)), and the adjoint through
<P x, y> = <x, P^T y> (2e-5 of the products' absolute sum)."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [(WALL, PERIODIC), (PERIODIC, WALL)])
@pytest.mark.parametrize("nx,ny,nz", [(18, 9, 3), (64, 8, 128), (54, 9, 129), (64, 16, 256), (36, 9, 257),
                                      (96, 8, 384), (54, 16, 385), (64, 9, 512)])
def test_fp32_z_lines(nx, ny, nz, bc):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(nx, ny, nz, *bc, lx=4.0, ly=4.0, lz=6.5, stretch=1.5)
    g = torch.Generator(device="cuda").manual_seed(nx + ny + nz)
    q = [torch.randn(spec.shape, dtype=torch.float64, device="cuda", generator=g) for _ in range(6)]
    for t in (q[:3], q[3:]):
        for a, m in zip(t, W.dead_face_masks(spec)):
            a[torch.from_numpy(m).cuda()] = 0.0
    p32, p64 = F.Plan.from_spec(spec, precision=F.PREC_FP32), F.Plan.from_spec(spec)
    x, y = [a.float() for a in q[:3]], [a.float() for a in q[3:]]
    px = [a.clone() for a in x]
    ref = [a.double() for a in x]
    p, r = p32.project(*px, dt=0.7), p64.project(*ref, dt=0.7)
    for a, b in zip([*px, p], [*ref, r]):
        assert float((a.double() - b).norm() / b.norm()) <= 2e-4
    pty = [a.clone() for a in y]
    p32.project_backward(*pty, None, dt=0.7)
    lhs = sum(float((a.double() * b.double()).sum()) for a, b in zip(px, y))
    rhs = sum(float((a.double() * b.double()).sum()) for a, b in zip(x, pty))
    scale = sum(float((a.double() * b.double()).abs().sum()) for a, b in zip(px, y))
    assert abs(lhs - rhs) <= 2e-5 * scale
