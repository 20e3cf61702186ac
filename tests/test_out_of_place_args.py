"""Out-of-place projection and adjoint refuse outputs that share memory with
another component's input, another output or p, before anything is launched
(no workspace here, no GPU): FSEI_ERR_ARG where the arrays overlap, and the
workspace error of an otherwise valid call where they do not.  In-place calls
take what they took before."""
import ctypes
import os

import pytest

from paper_2103_15187_amd import fsei
from test_abi_cpu import ERR_ARG, ERR_WORKSPACE, OK, create

pytestmark = pytest.mark.skipif(not os.path.exists(fsei.LIB_PATH), reason="libfsei.so not built")

NX, NY, NZ = 8, 6, 4
BASE = 1 << 20


@pytest.mark.parametrize("elem", [8, 4])
def test_overlapping_outputs(elem):
    L = fsei.lib()
    st, h = create(NX, NY, NZ)
    assert st == OK
    assert L.fsei_plan_set_precision(h, fsei.PREC_FP32 if elem == 4 else fsei.PREC_FP64, 1e-10, 4) == OK
    size = NX * NY * NZ * elem
    f = [ctypes.c_void_p(BASE + i * size) for i in range(8)]      # arrays side by side
    mid = ctypes.c_void_p(BASE + size // 2)                       # in the middle of f[0] and f[1]

    def fwd(u, v, w, ou, ov, ow, p):
        if elem == 4:
            return L.fsei_project_to_f32(h, u, v, w, ou, ov, ow, p, 1.0)
        return L.fsei_project_to(h, u, v, w, ou, ov, ow, p, 1.0, None)

    def bwd(gu, gv, gw, gp, ou, ov, ow):
        return (L.fsei_project_backward_to_f32 if elem == 4 else L.fsei_project_backward_to)(
            h, gu, gv, gw, gp, ou, ov, ow, 1.0)
    u, v, w, a, b, c, p, q = f
    # valid: apart, in place, some of each, no p, gp anywhere
    for args in ((u, v, w, a, b, c, p), (u, v, w, u, v, w, p), (u, v, w, u, b, w, p), (u, v, w, a, b, c, None)):
        assert fwd(*args) == ERR_WORKSPACE, args
    for args in ((u, v, w, p, a, b, c), (u, v, w, p, u, v, w), (u, v, w, None, a, b, c), (u, v, w, a, a, b, c)):
        assert bwd(*args) == ERR_WORKSPACE, args
    # an output on another input, on another output, across an input's end; p on an input or output
    for out in ((v, b, c), (a, w, c), (a, b, u), (a, a, c), (a, b, a), (mid, b, c), (a, mid, c)):
        assert fwd(u, v, w, *out, p) == ERR_ARG, out
        assert bwd(u, v, w, None, *out) == ERR_ARG, out
    for pp in (u, w, a, c, mid):
        assert fwd(u, v, w, a, b, c, pp) == ERR_ARG, pp
    # in place: as before
    d = ctypes.c_void_p(0x1000)
    if elem == 4:
        assert L.fsei_project_f32(h, d, d, d, d, 1.0) == ERR_WORKSPACE
        assert L.fsei_project_backward_f32(h, d, d, d, None, 1.0) == ERR_WORKSPACE
    else:
        assert L.fsei_project(h, d, d, d, d, 1.0, None) == ERR_WORKSPACE
        assert L.fsei_project_backward(h, d, d, d, None, 1.0) == ERR_WORKSPACE
    # null arguments and no plan
    assert fwd(u, v, w, None, b, c, p) == ERR_WORKSPACE
    assert L.fsei_project_to(None, u, v, w, a, b, c, p, 1.0, None) == ERR_ARG
    L.fsei_poisson_plan_destroy(h)
