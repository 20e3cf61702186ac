"""Refined solves whose x tiles outnumber the workspace's partial sums (lines
beyond 768, ny no multiple of 4, at most one near-singular line): the residual
passes take the kernel whose tiles run on across planes.  A sum left out or
written past its room would show in the residual, which is checked by the
oracle's stencil (<= 1e-10, the requested one), and in p and the velocities
against the FP64 solve, to the residual times the 1e4 that bounds the
condition of lines that are not near-singular."""
import pytest

import oracle
from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W
from test_gpu_parity import grid_of, rel, run_project

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(864, 9, 16), (972, 27, 5), (1024, 6, 16)])
@pytest.mark.parametrize("bc", [(WALL, PERIODIC), (PERIODIC, WALL)])
def test_refinement_without_room_for_every_tile(dims, bc):
    from paper_2103_15187_amd import fsei as F
    spec = W.small_spec(*dims, *bc, lx=1.0, ly=1.0, lz=50.0, stretch=1.0)
    g = grid_of(spec)
    u, v, w = W.random_velocity(spec, sum(dims))
    ref = run_project(spec, u, v, w)[:4]
    *got, info = run_project(spec, u, v, w, precision=F.PREC_FP32_REFINE, rtol=1e-10, max_iter=6)
    assert info["rel_residual"] <= 1e-10
    assert oracle.rel_residual(oracle.divergence(u, v, w, g), got[3], g) <= 1e-10
    for a, b in zip(got, ref):
        assert rel(a, b) <= 1e-6
