"""Near-singular lines in a launch of their own (more than one group per CU) on
short z lines: the number of chunks follows the length.  Parity on both sides
of each chunk count (bar 1e-12, rounding of at most 256 positive-factor steps
per line), and short lines that take less time than long ones."""
import pytest

from oracle import PERIODIC, WALL
from paper_2103_15187_amd import workloads as W
from test_gpu_parity import dev, grid_of, host, rel
from test_gpu_special_lines import _reference, _spec

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [4, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 256])
def test_parity_by_chunk_count(nz):
    from paper_2103_15187_amd import fsei as F
    spec = _spec(128, 64, nz, (WALL, PERIODIC))
    f = W.rng(nz).standard_normal(spec.shape)
    plan = F.Plan.from_spec(spec)
    plan.set_timing(True)
    p = plan.poisson_solve(dev(f))
    assert "zsolve_fp64_lines" in plan.kernel_times()
    e = rel(host(p), _reference(f, grid_of(spec)))
    print(nz, e)
    assert e <= 1e-12


def test_short_lines_take_less_time():
    # 262 thousand lines of 8 and of 64 rows: an eighth of the rows, at most half the time
    from paper_2103_15187_amd import fsei as F

    def best(nz):
        plan = F.Plan.from_spec(_spec(512, 512, nz, (WALL, PERIODIC)))
        f = torch.randn(plan.shape, dtype=torch.float64, device="cuda")
        ms = []
        plan.set_timing(True)
        for _ in range(6):
            plan.reset_timing()
            plan.poisson_solve(f)
            ms.append(plan.kernel_times()["zsolve_fp64_lines"][0])
        return min(ms)
    short, long = best(8), best(64)
    print(short, long)
    assert short <= 0.5 * long
