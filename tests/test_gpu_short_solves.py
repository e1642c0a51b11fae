"""Solves of one or two cycles or iterations launch about as many: the host looks at the
residual after the first cycle, and never launches more than the call allows.  Times are
medians; a call of one cycle may take three times the cycle itself (launching a batch of
eight took five to six times as long), and one CG iteration six times (it makes two
cycles; a batch of sixteen took over ten times as long).
"""
import time

import pytest

from meshgen import box_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _median(f, reps=15):
    times = []
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        f()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    return sorted(times)[reps // 2]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_one_cycle_costs_about_one_cycle(precision):
    from paper_2512_22215_amd import LduMatrix
    c = box_case(32, 32, 32, coeff="lognormal", dirichlet_x0=1.0, seed=3)
    m = LduMatrix.from_case(c)
    b = torch.from_numpy(c.rhs[0]).cuda()
    m.gamg_setup()
    cap = "max_refine" if precision == "mixed" else "max_cycles"

    def solve(cycles, tol):
        return m.gamg(b, rel_tol=tol, precision=precision, **{cap: cycles})
    x1, s1 = solve(1, 0.0)
    x2, s2 = solve(2, 0.0)
    assert (s1.iterations, s2.iterations) == (1, 2) and not torch.equal(x1, x2)
    cycle = _median(lambda: m.vcycle(b))
    assert _median(lambda: solve(1, 0.0)) <= 3.0 * cycle
    assert _median(lambda: solve(200, 0.5)) <= 3.0 * cycle  # stops after one
    m.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_one_iteration_costs_about_one_iteration(precision):
    from paper_2512_22215_amd import LduMatrix
    c = box_case(64, 64, 64, coeff="lognormal", dirichlet_x0=1.0, seed=3)
    m = LduMatrix.from_case(c)
    b = torch.from_numpy(c.rhs[0]).cuda()
    sweeps = dict(n_pre=1, n_post=1)
    m.gamg_setup(**sweeps)
    cap = dict(inner_max_iter=1, max_refine=1) if precision == "mixed" else dict(max_iter=1)
    _, s = m.pcg(b, precond=2, rel_tol=0.0, precision=precision, **cap)
    assert s.iterations == 1
    cycle = _median(lambda: m.vcycle(b, scale_correction=0, **sweeps))
    assert _median(lambda: m.pcg(b, precond=2, rel_tol=0.0, precision=precision, **cap)) <= 6 * cycle
    m.close()
