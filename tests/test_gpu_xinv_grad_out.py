"""The fused x inverse + gradient out of place, as autograd takes it, with
gradients of all four results (dLoss/dp among them), on grids large enough for
it: the same bits as the in-place calls on copies, the projection against the
plain 64-bit torch solve of perf/cases.py (bar 1e-12 relative L2, the FP64
path's), and the adjoint by <J x, y> = <x, J^T y> (bar 1e-12 of the products).
The adjoint's values by themselves are no measure of it: with dLoss/dp its u
and v are 30000 times smaller than the terms they are differences of."""
import pytest

from perf import cases

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,bc", [((256, 256, 261), "WP"), ((512, 512, 131), "PP"), ((576, 256, 257), "PW"),
                                     ((768, 256, 259), "WW")])
def test_autograd_takes_the_fused_kernel(dims, bc):
    case = dict(zip(("nx", "ny", "nz"), dims), kind="grad", bc=bc, prec="fp64", stretch=2.0, markers=0)
    assert dims[1] // 8 * dims[2] >= 32 * torch.cuda.get_device_properties(0).multi_processor_count
    s = cases.prepare(case, 5)
    plan, dt = s["plan"], s["dt"]
    keep = [s[k].detach().clone() for k in "uvw"]
    weights = [t.clone() for t in s["weights"]]
    plan.set_timing(True)
    got = cases.run(s)
    assert plan.kernel_times()["xinv_grad"][1] == 2 and "grad" not in plan.kernel_times()
    plan.set_timing(False)
    assert all(torch.equal(s[k].detach(), a) for k, a in zip("uvw", keep))
    assert all(torch.equal(a, b) for a, b in zip(s["weights"], weights))
    q = [a.clone() for a in keep]
    q.append(plan.project(*q, dt=dt))
    assert all(torch.equal(a, b) for a, b in zip(got["out"], q))
    plan.project_backward(*weights, dt=dt)
    assert all(torch.equal(a, b) for a, b in zip(got["grad"], weights))
    for a, b in zip(got["out"], cases.exact(case, 5)["out"]):
        assert float((a - b).norm() / b.norm()) <= 1e-12
    # the inputs' dead wall faces are 0, so <J x, y> = <x, J^T y>
    lhs = sum(float((a * b).sum()) for a, b in zip(got["out"], s["weights"]))
    rhs = sum(float((a * b).sum()) for a, b in zip(keep, got["grad"]))
    scale = sum(float((a * b).abs().sum()) for a, b in zip(got["out"], s["weights"]))
    assert abs(lhs - rhs) <= 1e-12 * scale
