"""Diagonal CG and PBiCG at the sizes and layouts where their kernels change: just below
and above the cells up to which an iteration is two kernels (160,000 for CG, 65,536 for
PBiCG), one slice and less, a random numbering (32-bit columns), rows of uneven length
(compressed slices).  Bars as in the parity tests: equal iteration counts, histories to
1e-9 and solutions to 1e-10 for CG, counts within one and 1e-8 for PBiCG, against the
oracle; CG without a preconditioner only follows the oracle's rounding for its first 20
iterations on these systems, and is held to its true residual after that.  How often the
host looks at the scalars must not change a bit.
"""
import numpy as np
import pytest

import oracle as O
from meshgen import LduCase, assemble_diag, box_case, random_order, relabel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _uneven(n, nonsym):
    """A chain with random extra faces: row lengths from 2 to about 20."""
    rng = np.random.default_rng(n)
    hub = rng.integers(0, n // 8, 4 * n)
    far = rng.integers(0, n, 4 * n)
    pairs = {(i, i + 1) for i in range(n - 1)}
    pairs |= {(min(a, b), max(a, b)) for a, b in zip(hub, far) if a != b}
    own, nb = np.array(sorted(pairs), np.int32).T
    up = np.exp(0.5 * rng.standard_normal(own.size))
    lo = up * np.exp(nonsym * rng.standard_normal(own.size)) if nonsym else up.copy()
    big = np.maximum(up, lo)
    diag = assemble_diag(n, own, nb, big, big, np.full(n, 0.5))
    return LduCase("uneven", n, own, nb, diag, up, lo, [rng.standard_normal(n)])


def _case(name, nonsym):
    if name == "uneven":
        return _uneven(3000, nonsym)
    dims = {"one-slice": (5, 4, 3), "two-slices": (13, 5, 1), "random": (41, 37, 29),
            "cg-below": (54, 54, 54), "cg-above": (55, 54, 54),
            "bicg-below": (41, 40, 39), "bicg-above": (41, 40, 40)}[name]
    c = box_case(*dims, coeff="lognormal", dirichlet_x0=1.0, nonsym=nonsym, seed=11)
    return relabel(c, random_order(c.n_cells, np.random.default_rng(12))) \
        if name == "random" else c


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("precond", [0, 1])
@pytest.mark.parametrize("name", ["one-slice", "two-slices", "random", "uneven", "cg-below",
                                  "cg-above"])
def test_cg_steps(name, precond):
    from paper_2512_22215_amd import LduMatrix
    c = _case(name, 0.0)
    m = LduMatrix.from_case(c)
    if name in ("uneven", "cg-above"):  # one of each layout
        assert m.layout(0)["compressed"] == (name == "uneven")
    tol = 1e-8 if c.n_cells < 100000 else 1e-3
    ref = O.pcg(O.Ldu.from_case(c), c.rhs[0], tol=tol, precond=bool(precond))
    xs = []
    for every in (16, 5, 1):
        x, st = m.pcg(_t(c.rhs[0]), rel_tol=tol, precond=precond, check_every=every,
                      history=2000)
        xs.append(x.cpu().numpy())
        assert st.converged
        h = np.asarray(st.history)
        if precond:
            assert st.iterations == ref.iterations
            assert np.all(np.abs(h - ref.history) <= 1e-9 * ref.history + 1e-15)
            assert np.linalg.norm(xs[-1] - ref.x) <= 1e-10 * np.linalg.norm(ref.x)
        else:  # both sides lose orthogonality: the histories part after some 30 iterations
            assert np.all(np.abs(h[:21] - ref.history[:21]) <= 1e-9 * ref.history[:21])
            r = c.rhs[0] - O.amul(O.Ldu.from_case(c), xs[-1])
            assert np.linalg.norm(r) <= tol * np.linalg.norm(c.rhs[0]) * (1 + 1e-6)
    assert np.array_equal(xs[0], xs[1]) and np.array_equal(xs[0], xs[2])
    m.close()


@pytest.mark.parametrize("precond", [0, 1])
@pytest.mark.parametrize("name", ["one-slice", "two-slices", "random", "uneven",
                                  "bicg-below", "bicg-above"])
def test_pbicg_steps(name, precond):
    from paper_2512_22215_amd import LduMatrix
    c = _case(name, 0.4)
    A = O.Ldu.from_case(c)
    m = LduMatrix.from_case(c)
    if name in ("uneven", "bicg-above"):
        assert m.layout(0)["compressed"] == (name == "uneven")
    for solve, tr in ((m.pbicg, False), (lambda *a, **k: m.adjoint(*a, solver="pbicg", **k),
                                         True)):
        ref = O.pbicg(A, c.rhs[0], tol=1e-8, precond=bool(precond), transpose=tr)
        xs = []
        for every in (16, 3):
            x, st = solve(_t(c.rhs[0]), rel_tol=1e-8, precond=precond, check_every=every)
            assert st.converged and abs(st.iterations - ref.iterations) <= 1
            xs.append(x.cpu().numpy())
            assert np.linalg.norm(xs[-1] - ref.x) <= 1e-8 * np.linalg.norm(ref.x)
        assert np.array_equal(xs[0], xs[1])
    m.close()
