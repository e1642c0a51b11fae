"""Jacobi cycles without the one-pass down leg (several pre-sweeps, scaled corrections) on
small levels, whose sweeps, restriction and up leg share rows between lanes: every
combination of sweeps up to three, scaled or not, against the oracle's separate steps, on
a chain (short rows), boxes, merged aggregates (long rows), a level 0 at and just above
the 65,536 cells up to which the path runs; new coefficients and relaxation factors; A^T;
the FP32 cycle inside refinement; CG with a symmetric cycle of two sweeps.  The bar is the
V-cycle bar of the parity tests, 1e-11: the same terms summed in a different order.
"""
import numpy as np
import pytest

import oracle as O
from meshgen import box_case, random_order, relabel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "chain": (dict(nx=300, ny=1, nz=1), {}),
    "box": (dict(nx=19, ny=17, nz=13), {}),
    "merged": (dict(nx=23, ny=21, nz=11), dict(passes=3, aggressive_from=0)),
    "at-limit": (dict(nx=64, ny=64, nz=16), {}),
    "above-limit": (dict(nx=241, ny=17, nz=16), {}),
}


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _close(x, ref, tol):
    return np.linalg.norm(x.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("nonsym", [0.0, 0.5])
@pytest.mark.parametrize("name", list(CASES))
def test_small_level_cycles(name, nonsym):
    from paper_2512_22215_amd import LduMatrix
    dims, hier = CASES[name]
    c = box_case(**dims, coeff="lognormal", dirichlet_x0=1.0, nonsym=nonsym, seed=51)
    if name == "box":
        c = relabel(c, random_order(c.n_cells, np.random.default_rng(52)))
    A = O.Ldu.from_case(c)
    m = LduMatrix.from_case(c)
    g = O.Gamg(A, **hier)
    r = np.random.default_rng(53).standard_normal(c.n_cells)

    def check(n_pre, n_post, scale, omega=0.75):
        e = m.vcycle(_t(r), n_pre=n_pre, n_post=n_post, scale_correction=int(scale),
                     omega=omega, **hier)
        assert _close(e, g.vcycle(r, n_pre=n_pre, n_post=n_post, omega=omega, scale=scale),
                      1e-11), (n_pre, n_post, scale, omega)

    for n_pre, n_post in ((1, 1), (2, 2), (3, 1), (1, 3)):
        check(n_pre, n_post, True)
    check(2, 2, False)
    check(2, 1, False)
    check(2, 2, True, omega=0.6)
    m.set_coeffs(_t(2.0 * c.diag), _t(c.upper), _t(0.5 * c.lower))
    g.set_values(2.0 * c.diag, c.upper, 0.5 * c.lower)
    check(2, 2, True, omega=0.6)
    check(2, 2, True)
    m.set_coeffs(_t(c.diag), _t(c.upper), _t(c.lower))
    g.set_values(c.diag, c.upper, c.lower)
    b = c.rhs[0]
    for tr in (False, True):
        opts = dict(rel_tol=0.0, max_cycles=3, **hier)
        x = m.adjoint(_t(b), solver="gamg", **opts)[0] if tr else m.gamg(_t(b), **opts)[0]
        assert _close(x, g.solve(b, tol=0.0, max_cycles=3, transpose=tr).x, 1e-10)
    if nonsym == 0.0:
        x, st = m.gamg(_t(b), rel_tol=1e-10, precision="mixed", max_refine=400, **hier)
        res = b - O.amul(A, x.cpu().numpy())
        assert st.converged and np.linalg.norm(res) <= 1.001e-10 * np.linalg.norm(b)
        m.gamg_setup(**hier)  # CG with the default two sweeps each way
        for solve, tr in ((m.pcg, False), (m.adjoint, True)):
            x, st = solve(_t(b), precond=2, rel_tol=1e-8)
            ref = g.pcg(b, tol=1e-8, transpose=tr)
            assert st.converged and st.iterations == ref.iterations
            assert _close(x, ref.x, 1e-9)
    m.close()
