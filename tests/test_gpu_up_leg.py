"""The up leg of small levels as one operator, e = U (r, e_c): V-cycles with one
Jacobi pre-sweep and no correction scaling, against the oracle's separate steps (first
sweep, correction, post-sweep), at the sizes where the path or the lanes per row change:
a chain (short rows, short rows on the coarsest level too), level 0 at and just above the
65,536 cells up to which it runs through U, merged aggregates (long rows), one and two
post-sweeps, two relaxation factors, new coefficients, A^T.

The bar is the V-cycle bar of the parity tests, 1e-11 relative: both sides sum the same
terms in a different order, a few hundred roundings of 1e-16 each per row and level.
"""
import numpy as np
import pytest

import oracle as O
from meshgen import box_case, random_order, relabel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MERGED = dict(passes=3, aggressive_from=0)
CASES = {
    "chain": (dict(nx=400, ny=1, nz=1), {}, 1),
    "pairwise": (dict(nx=23, ny=19, nz=17), {}, 1),
    "pairwise-two-post": (dict(nx=23, ny=19, nz=17), {}, 2),
    "merged": (dict(nx=31, ny=29, nz=13), MERGED, 1),
    "at-limit": (dict(nx=64, ny=64, nz=16), {}, 1),
    "above-limit": (dict(nx=241, ny=17, nz=16), {}, 1),
}


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("nonsym", [0.0, 0.5])
def test_up_leg_operator(name, nonsym):
    from paper_2512_22215_amd import LduMatrix
    dims, hier, n_post = CASES[name]
    c = box_case(**dims, coeff="lognormal", dirichlet_x0=1.0, nonsym=nonsym, seed=31)
    if name == "pairwise":
        c = relabel(c, random_order(c.n_cells, np.random.default_rng(32)))
    assert (c.n_cells <= 1 << 16) == (name != "above-limit")
    m = LduMatrix.from_case(c)
    g = O.Gamg(O.Ldu.from_case(c), **hier)
    r = np.random.default_rng(33).standard_normal(c.n_cells)
    cycle = dict(n_pre=1, n_post=n_post, scale_correction=0, **hier)

    def check(omega):
        e = m.vcycle(_t(r), omega=omega, **cycle).cpu().numpy()
        ref = g.vcycle(r, n_pre=1, n_post=n_post, omega=omega, scale=False)
        assert np.linalg.norm(e - ref) <= 1e-11 * np.linalg.norm(ref), omega

    for omega in (0.75, 0.6, 0.75):
        check(omega)
    # A^T, through the adjoint solve with the cycle as CG's preconditioner, and r.z
    # taken by the up leg of level 0 when that level is small
    if nonsym == 0.0 and n_post == 1:
        m.gamg_setup(**cycle)
        for solve, tr in ((m.pcg, False), (m.adjoint, True)):
            x, st = solve(_t(c.rhs[0]), precond=2, rel_tol=1e-8)
            ref = g.pcg(c.rhs[0], tol=1e-8, n_pre=1, n_post=1, transpose=tr)
            assert st.converged and st.iterations == ref.iterations
            assert (np.linalg.norm(x.cpu().numpy() - ref.x)
                    <= 1e-9 * np.linalg.norm(ref.x))
    else:
        ref = g.solve(c.rhs[0], tol=0.0, max_cycles=3, n_pre=1, n_post=n_post, scale=False,
                      transpose=True)
        x, _ = m.adjoint(_t(c.rhs[0]), solver="gamg", rel_tol=0.0, max_cycles=3, **cycle)
        assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    # new coefficients on the kept hierarchy
    m.set_coeffs(_t(2.0 * c.diag), _t(c.upper), _t(0.5 * c.lower))
    g.set_values(2.0 * c.diag, c.upper, 0.5 * c.lower)
    check(0.75)
    m.close()
