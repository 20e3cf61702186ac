"""Viscous x solves with two and with four tiles per workgroup and a ragged last
workgroup (one workgroup per CU: 768 rows) against the oracle; bar 1e-12 of
max |oracle|, as for the other line lengths."""
import numpy as np
import pytest

from oracle import PERIODIC, WALL
from oracle import viscous as V
from paper_2103_15187_amd import workloads as W
from test_gpu_viscous import dev, grid_of, host

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bcx", [WALL, PERIODIC])
@pytest.mark.parametrize("dims", [(768, 27, 147), (768, 81, 97)])
def test_tiles_per_workgroup(dims, bcx):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(*dims, bcx, PERIODIC, lx=4.0, ly=4.0, lz=6.5, stretch=1.5)
    g, beta = grid_of(spec), 3.0 * spec.dx ** 2
    r = W.rng(sum(dims)).standard_normal(spec.shape)
    q = dev(r)
    F.Plan.from_spec(spec).viscous_solve(q, 0, beta)
    ref = V.viscous_solve(r, g, 0, beta)
    assert np.abs(host(q) - ref).max() <= 1e-12 * np.abs(ref).max()
