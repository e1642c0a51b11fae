"""Setup kernels that share a row between lanes, at the row lengths where they change
path: complete graphs, whose rows hold every other cell.  9 and 10 cells sit at the edge
of the in-register sort of lower entries (8), 17 and 18 at one and two passes of a coarse
row's 16 lanes, 65 and 66 at one and two passes of a wave, 130 above the 256 candidates a
coarse row holds in LDS, 255 (an odd count: one aggregate of three) above the 512 pairs a
restriction row does.  A chain of 1200 cells has the shortest rows.

Integer results and Galerkin values equal the oracle's bit for bit (the same sums in the
same order); V-cycles meet the parity tests' bar of 1e-11.
"""
import numpy as np
import pytest

import oracle as O
from meshgen import LduCase, assemble_diag, box_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _complete(n):
    own, nb = np.triu_indices(n, 1)
    rng = np.random.default_rng(n)
    a = np.exp(rng.standard_normal(own.size))
    lo = a * np.exp(0.2 * rng.standard_normal(own.size))
    diag = 1.3 * assemble_diag(n, own, nb, np.maximum(a, lo), np.maximum(a, lo))
    return LduCase("complete", n, own.astype(np.int32), nb.astype(np.int32), diag, a, lo,
                   [rng.standard_normal(n)])


@pytest.mark.parametrize("passes", [1, 2])
@pytest.mark.parametrize("n", [9, 10, 17, 18, 65, 66, 130, 255, -1200])
def test_setup_row_lengths(n, passes):
    from paper_2512_22215_amd import LduMatrix
    c = _complete(n) if n > 0 else box_case(-n, 1, 1, coeff="lognormal", dirichlet_x0=1.0,
                                            seed=3)
    A = O.Ldu.from_case(c)
    m = LduMatrix.from_case(c)
    x = np.random.default_rng(5).standard_normal(c.n_cells)
    assert np.array_equal(m.amul(x).cpu().numpy(), O.amul(A, x))
    assert np.array_equal(m.tmul(x).cpu().numpy(), O.tmul(A, x))
    g = O.Gamg(A, n_coarsest=4, passes=passes)
    cycle = dict(n_pre=1, n_post=1, scale_correction=0, n_coarsest=4, passes=passes)
    m.gamg_setup(**cycle)
    assert m.n_levels() == g.n_levels > 1
    for lev in range(g.n_levels):
        got, ref = m.level(lev), g.level(lev)
        assert (got["n"], got["nf"]) == (ref.n, ref.nf)
        if ref.agg is not None:
            assert np.array_equal(got["agg"].cpu().numpy(), ref.agg)
        for key, want in (("owner", ref.owner), ("neighbour", ref.neighbour),
                          ("diag", ref.diag), ("upper", ref.upper), ("lower", ref.lower)):
            assert np.array_equal(got[key].cpu().numpy(), want), (lev, key)
    for scale in (0, 1):  # with and without the one-pass down leg
        e = m.vcycle(x, **dict(cycle, scale_correction=scale)).cpu().numpy()
        ref = g.vcycle(x, n_pre=1, n_post=1, scale=bool(scale))
        assert np.linalg.norm(e - ref) <= 1e-11 * np.linalg.norm(ref)
    m.close()
