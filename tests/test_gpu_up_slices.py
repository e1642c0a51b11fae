"""The up leg of a large plain-slice level (scaled slices) in one pass, from the down
leg's t and the coarse vector, against the oracle's separate steps (first sweep,
correction, post-sweeps): a box whose last slice is ragged and whose planes are so large
that some slices span more than 65,535 aggregates, symmetric and not, one post-sweep
(which takes r.z in the CG) and two, A^T, the mixed form.

The bars are those of the parity tests for the same cycles: 1e-11 relative for a V-cycle
(both sides sum the same terms in a different order), 1e-9 for a solution, 1e-10 for the
true residual of the mixed form.
"""
import numpy as np
import pytest

import oracle as O
from meshgen import box_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("nonsym", [0.0, 0.5])
@pytest.mark.parametrize("n_post", [1, 2])
def test_up_leg_from_scaled_slices(nonsym, n_post):
    from paper_2512_22215_amd import LduMatrix
    c = box_case(400, 401, 5, coeff="lognormal", dirichlet_x0=1.0, nonsym=nonsym, seed=51)
    cycle = dict(n_pre=1, n_post=n_post, scale_correction=0)
    m = LduMatrix.from_case(c)
    m.gamg_setup(**cycle)
    g = O.Gamg(O.Ldu.from_case(c))
    assert c.n_cells % 64 != 0 and m.downleg(0) == ("scaled_slices", 0)
    r = np.random.default_rng(52).standard_normal(c.n_cells)
    for omega in (0.75, 0.6):
        e = m.vcycle(_t(r), omega=omega, **cycle).cpu().numpy()
        ref = g.vcycle(r, n_pre=1, n_post=n_post, omega=omega, scale=False)
        assert np.linalg.norm(e - ref) <= 1e-11 * np.linalg.norm(ref), omega
    b = c.rhs[0]
    m.gamg_setup(**cycle)
    if nonsym:
        x, _ = m.adjoint(_t(b), solver="gamg", rel_tol=0.0, max_cycles=2, **cycle)
        ref = g.solve(b, tol=0.0, max_cycles=2, n_pre=1, n_post=n_post, scale=False,
                      transpose=True)
        assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
    else:
        x, st = m.pcg(_t(b), precond=2, rel_tol=1e-8)
        ref = g.pcg(b, tol=1e-8, n_pre=1, n_post=n_post)
        assert st.converged and st.iterations == ref.iterations
        assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-9 * np.linalg.norm(ref.x)
        x, st = m.pcg(_t(b), precond=2, rel_tol=1e-10, precision="mixed")
        true = O.amul(O.Ldu.from_case(c), x.cpu().numpy())
        assert st.converged
        assert np.linalg.norm(b - true) <= 1e-10 * np.linalg.norm(b) * 1.01
    m.close()
