"""PBiCG on compressed slices (rows of uneven length), with a matrix that stays in the
Infinity Cache between two products and with one that streams past it, against the oracle:
equal counts and solutions within 1e-9, forward and transposed.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _band(n):
    """One to five upper neighbours a cell within some 40 cells; upwind coefficients."""
    rng = np.random.default_rng(n)
    own = np.repeat(np.arange(n, dtype=np.int64), rng.integers(1, 6, n))
    nb = own + rng.integers(1, 40, own.size)
    own, nb = own[nb < n], nb[nb < n]
    key = np.unique(own * n + nb)
    own, nb = (key // n).astype(np.int32), (key % n).astype(np.int32)
    upper = -rng.uniform(0.5, 1.0, own.size)
    lower = 1.3 * upper
    diag = 0.5 - np.bincount(own, lower, n) - np.bincount(nb, lower, n)
    return n, own, nb, diag, upper, lower


@pytest.mark.parametrize("n", [1, 63, 700, 20000, 1500000])
def test_pbicg_on_uneven_rows(n):
    from paper_2512_22215_amd import LduMatrix
    a = _band(n)
    m = LduMatrix(a[0], *map(_t, a[1:]))
    if n >= 700:
        assert m.layout(0)["compressed"]
    b = np.random.default_rng(7).standard_normal(n)
    A = O.Ldu(*a)
    for solve, tr in ((m.pbicg, False), (lambda v, **k: m.adjoint(v, solver="pbicg", **k), True)):
        x, st = solve(_t(b), rel_tol=1e-10)
        ref = O.pbicg(A, b, tol=1e-10, transpose=tr)
        assert st.converged and st.iterations == ref.iterations
        assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-9 * np.linalg.norm(ref.x)
    m.close()
