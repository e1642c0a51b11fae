"""U's values, formed by 16 lanes a row, on rows with few and with many aggregates: a
chain whose first cell is also joined to `spokes` others, so that its row on level 0
holds up to 16, 32 and 64 aggregates (one to four to a lane) and more (formed by one
lane), against the oracle's separate steps, for two relaxation factors and new
coefficients.

The bar is the V-cycle bar of the parity tests, 1e-11 relative.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("spokes", [0, 14, 40, 100])
def test_up_rows_of_any_length(spokes):
    from paper_2512_22215_amd import LduMatrix
    n = 997
    rng = np.random.default_rng(61)
    faces = {(i, i + 1) for i in range(n - 1)} | {(0, 3 * k) for k in range(1, spokes + 1)}
    own, nb = (np.array(a, np.int32) for a in zip(*sorted(faces)))
    upper = -rng.uniform(0.5, 1.5, len(own))
    lower = upper * rng.uniform(0.8, 1.2, len(own))
    diag = np.full(n, 0.05)
    np.subtract.at(diag, own, upper)
    np.subtract.at(diag, nb, lower)
    m = LduMatrix(n, *map(_t, (own, nb, diag, upper, lower)))
    g = O.Gamg(O.Ldu(n, own, nb, diag, upper, lower))
    r = rng.standard_normal(n)

    def check(omega):
        e = m.vcycle(_t(r), omega=omega, n_pre=1, n_post=1, scale_correction=0).cpu().numpy()
        ref = g.vcycle(r, n_pre=1, n_post=1, omega=omega, scale=False)
        assert np.linalg.norm(e - ref) <= 1e-11 * np.linalg.norm(ref), omega

    for omega in (0.75, 0.6):
        check(omega)
    m.set_coeffs(_t(2.0 * diag), _t(upper), _t(0.5 * lower))
    g.set_values(2.0 * diag, upper, 0.5 * lower)
    check(0.6)
    m.close()
