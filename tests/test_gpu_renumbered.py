"""Solves on a mesh whose numbering scatters its neighbours (a random one, above the
500,000 cells from which the hierarchy's large levels are renumbered for the solves):
everything in the caller's numbering stays exact (products, hierarchy), and V-cycles,
GAMG, CG + V-cycle and the mixed form, forward and transposed, with new coefficients and
with the two-stage Gauss-Seidel smoother (which keeps the original numbering) meet the
parity tests' bars against the oracle: V-cycles to 1e-11, equal counts, solutions to 1e-9.
A mesh just below the limit and one in natural order go through the same checks.
"""
import numpy as np
import pytest

import oracle as O
from meshgen import box_case, random_order, relabel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HIER = {"pairwise": {}, "merged": dict(passes=3, aggressive_from=1)}


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _close(x, ref, tol):
    return np.linalg.norm(x.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("name,nonsym", [("shuffled", 0.0), ("shuffled", 0.4),
                                         ("below", 0.0), ("natural", 0.0)])
@pytest.mark.parametrize("hier", list(HIER))
def test_renumbered_levels(name, nonsym, hier):
    from paper_2512_22215_amd import LduMatrix
    c = box_case(83, 80 if name == "below" else 81, 75, coeff="lognormal", dirichlet_x0=1.0,
                 nonsym=nonsym, seed=41)
    assert (c.n_cells < 500000) == (name == "below")
    if name != "natural":
        c = relabel(c, random_order(c.n_cells, np.random.default_rng(42)))
    kw = HIER[hier]
    A = O.Ldu.from_case(c)
    m = LduMatrix.from_case(c)
    g = O.Gamg(A, **kw)
    one = dict(n_pre=1, n_post=1, **kw)
    m.gamg_setup(**one)
    b = c.rhs[0]
    assert np.array_equal(m.amul(b).cpu().numpy(), O.amul(A, b))
    assert m.n_levels() == g.n_levels
    for lev in range(g.n_levels):
        got, ref = m.level(lev), g.level(lev)
        if ref.agg is not None:
            assert np.array_equal(got["agg"].cpu().numpy(), ref.agg)
        assert np.array_equal(got["owner"].cpu().numpy(), ref.owner)
        assert np.array_equal(got["diag"].cpu().numpy(), ref.diag)
        assert np.array_equal(got["upper"].cpu().numpy(), ref.upper)

    def cycles():
        for cyc, ref in ((dict(one, scale_correction=0), dict(n_pre=1, n_post=1, scale=False)),
                         (kw, dict(n_pre=2, n_post=2, scale=True))):
            assert _close(m.vcycle(_t(b), **cyc), g.vcycle(b, **ref), 1e-11)

    cycles()
    if nonsym == 0.0:
        for tr in (False, True):
            solve = m.adjoint if tr else m.pcg
            m.gamg_setup(**one)
            x, st = solve(_t(b), precond=2, rel_tol=1e-8)
            ref = g.pcg(b, tol=1e-8, n_pre=1, n_post=1, transpose=tr)
            assert st.converged and st.iterations == ref.iterations
            assert _close(x, ref.x, 1e-9)
        x0 = np.random.default_rng(43).standard_normal(c.n_cells)
        x, st = m.pcg(_t(b), x0=_t(x0), precond=2, rel_tol=1e-10, precision="mixed")
        r = b - O.amul(A, x.cpu().numpy())
        assert st.converged and np.linalg.norm(r) <= 1.001e-10 * np.linalg.norm(b)
    for tr in (False, True):
        opts = dict(rel_tol=0.0, max_cycles=3, **kw)
        x = m.adjoint(_t(b), solver="gamg", **opts)[0] if tr else m.gamg(_t(b), **opts)[0]
        assert _close(x, g.solve(b, tol=0.0, max_cycles=3, transpose=tr).x, 1e-10)
    gs = O.Gamg(A, smoother="gs2", **kw)
    assert _close(m.vcycle(_t(b), smoother="gs2", **kw), gs.vcycle(b), 1e-11)
    d2, u2, l2 = 2.0 * c.diag, 1.5 * c.upper, 1.25 * c.lower
    m.set_coeffs(_t(d2), _t(u2), _t(l2))
    g.set_values(d2, u2, l2)
    cycles()
    m.close()
