"""The projection that keeps its input (fsei.project, fsei_project_to) and its
adjoint against the in-place entry points on copies: the same kernels on the
same values, so the same bits, and the inputs unchanged.  Inputs that the
kernels cannot read where they lie (strided, expanded, off the 16-byte
alignment) go through a copy and give the same result."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# every gradient kernel: fused x inverse, row pairs, odd rows, rows beyond 1024
SHAPES = [((512, 16, 6), (WALL, PERIODIC)), ((36, 24, 40), (PERIODIC, WALL)), ((27, 18, 20), (WALL, WALL)),
          ((1536, 9, 4), (PERIODIC, PERIODIC))]


def _plan(F, dims, bc, prec):
    spec = W.small_spec(*dims, *bc, lx=4.0, ly=4.0, lz=6.5, stretch=2.0)
    kw = {"fp64": {}, "fp32": dict(precision=F.PREC_FP32),
          "refine": dict(precision=F.PREC_FP32_REFINE, rtol=1e-10, max_iter=4, accept_floor=True)}[prec]
    return spec, F.Plan.from_spec(spec, **kw)


def _fields(spec, prec, seed, n=3):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dtype = torch.float32 if prec == "fp32" else torch.float64
    return [torch.randn(spec.shape, dtype=dtype, device="cuda", generator=g) for _ in range(n)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "refine"])
@pytest.mark.parametrize("dims,bc", SHAPES)
def test_same_as_in_place_and_inputs_kept(dims, bc, prec):
    from paper_2103_15187_amd import fsei as F
    spec, plan = _plan(F, dims, bc, prec)
    q = _fields(spec, prec, 3)
    ref = [t.clone() for t in q]
    ref.append(plan.project(*ref, dt=0.7))
    x = [t.clone().requires_grad_(True) for t in q]
    out = F.project(*x, plan, 0.7)
    for a, b, c, d in zip(out[:3], ref, x, q):
        assert torch.equal(a, b) and torch.equal(c, d)
    assert torch.equal(out[3], ref[3])
    gw = _fields(spec, prec, 5, 4)
    keep = [t.clone() for t in gw]
    grads = torch.autograd.grad(out, x, gw)
    gref = [t.clone() for t in gw[:3]]
    plan.project_backward(*gref, gw[3], dt=0.7)
    assert all(torch.equal(a, b) for a, b in zip(grads, gref))
    assert all(torch.equal(a, b) for a, b in zip(gw, keep))


@pytest.mark.parametrize("dims,bc", SHAPES[:3])
def test_inputs_that_need_a_copy(dims, bc):
    from paper_2103_15187_amd import fsei as F
    spec, plan = _plan(F, dims, bc, "fp64")
    u, v, w = _fields(spec, "fp64", 7)
    w = w[:1].expand(spec.shape)
    ref = F.project(u, v, w.contiguous(), plan, 0.7)
    off = torch.empty(u.numel() + 1, dtype=u.dtype, device="cuda")[1:].view(u.shape)
    off.copy_(u)
    assert off.data_ptr() % 16 == 8
    strided = torch.empty((*v.shape[:2], 2 * v.shape[2]), dtype=v.dtype, device="cuda")[:, :, ::2]
    strided.copy_(v)
    got = F.project(off, strided, w, plan, 0.7)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
    with pytest.raises(ValueError):   # dense but in another order: refused, as by the in-place call
        F.project(u.transpose(0, 2).contiguous().transpose(0, 2), v, w.contiguous(), plan, 0.7)
    # the loss's gradient as an expanded tensor
    x = u.clone().requires_grad_(True)
    gs = torch.autograd.grad(F.project(x, v, w.contiguous(), plan, 0.7)[0].sum(), x)[0]
    gu = torch.ones_like(u)
    plan.project_backward(gu, torch.zeros_like(u), torch.zeros_like(u), None, dt=0.7)
    assert float((gs - gu).norm() / gu.norm()) <= 1e-12
