"""Near-singular lines and zero mode inside the FP32 kernels of more than 1024
rows and of 769 to 1024 rows with nx odd (workgroups of 1024 threads, where the
threads beyond the first 512 repeat their work): the right-hand side is one
near-singular x mode times a z profile, so the first FP32 solve (no
correction) is that line alone.  Bar 1e-5: the transforms' FP32 rounding
(2^-24 times some ten steps) in modes that the solve amplifies less than this one."""
import numpy as np
import pytest

from oracle import WALL
from paper_2103_15187_amd import workloads as W
from test_gpu_parity import dev, grid_of, host, rel
from test_gpu_special_lines import _reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(27, 9, 300), (27, 9, 800), (27, 9, 1100), (27, 9, 1600), (54, 9, 640), (64, 8, 700),
                                  (32, 8, 1000), (32, 8, 1100), (32, 8, 1600), (32, 8, 2048), (54, 162, 200)])
def test_line_inside_fp32_kernels(dims):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(*dims, WALL, WALL, lx=40.0, ly=1.0, lz=6.5, stretch=1.5)
    dz = np.diff(spec.zc()).min()
    lam = 4.0 / spec.dx ** 2 * np.sin(np.pi / (2 * spec.nx)) ** 2
    assert lam < 4.0 / (dz * dz * 9999.0)              # mode (1, 0) is near-singular
    x = np.cos(np.pi * (np.arange(spec.nx) + 0.5) / spec.nx)
    f = W.rng(sum(dims)).standard_normal((spec.nz, 1, 1)) * np.ones((1, spec.ny, 1)) * x
    plan = F.Plan.from_spec(spec, precision=F.PREC_FP32_REFINE, rtol=0.0, max_iter=0)
    p = plan.poisson_solve(dev(np.ascontiguousarray(f)))
    e = rel(host(p), _reference(f, grid_of(spec)))
    print(dims, e)
    assert e <= 1e-5
