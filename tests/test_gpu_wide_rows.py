"""Cycles on levels with a wide row: a chain with one more cell that `spokes` of the others
are joined to, whose row lies in up to 64 aggregates (the most that the operators U and V
take) or more, and a star, whose one aggregate gathers more pairs than a restriction row
holds in LDS.  The bar is the V-cycle bar of the parity tests, 1e-11 relative.

A wide row keeps the cycle's time: formed entry by entry by one lane, the star's operators
took over a second.
"""
import time

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CYCLES = [dict(n_pre=2, n_post=2, scale_correction=1), dict(n_pre=1, n_post=2, scale_correction=1),
          dict(n_pre=1, n_post=1, scale_correction=0)]


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _matrix(n, faces, seed):
    own, nb = (np.array(a, np.int32) for a in zip(*sorted(faces)))
    rng = np.random.default_rng(seed)
    upper = -rng.uniform(0.5, 1.5, len(own))
    lower = upper * rng.uniform(0.8, 1.2, len(own))
    diag = np.full(n, 0.05)
    np.subtract.at(diag, own, upper)
    np.subtract.at(diag, nb, lower)
    return own, nb, diag, upper, lower


def _check(n, faces, seed):
    from paper_2512_22215_amd import LduMatrix
    own, nb, diag, upper, lower = _matrix(n, faces, seed)
    m = LduMatrix(n, *map(_t, (own, nb, diag, upper, lower)))
    g = O.Gamg(O.Ldu(n, own, nb, diag, upper, lower))
    r = np.random.default_rng(seed + 1).standard_normal(n)

    def check(omega):
        for c in CYCLES:
            e = m.vcycle(_t(r), omega=omega, **c).cpu().numpy()
            ref = g.vcycle(r, n_pre=c["n_pre"], n_post=c["n_post"], omega=omega,
                           scale=bool(c["scale_correction"]))
            assert np.linalg.norm(e - ref) <= 1e-11 * np.linalg.norm(ref), (omega, c)
    for omega in (0.75, 0.6):
        check(omega)
    m.set_coeffs(_t(2.0 * diag), _t(upper), _t(0.5 * lower))
    g.set_values(2.0 * diag, upper, 0.5 * lower)
    check(0.6)
    m.close()


@pytest.mark.parametrize("spokes", [15, 16, 62, 63, 64, 65, 120])
def test_cell_with_many_neighbours(spokes):
    n = 1500
    _check(n, {(i, i + 1) for i in range(n - 2)} | {(5 * k, n - 1) for k in range(spokes)}, 71)


@pytest.mark.parametrize("leaves", [100, 300])
def test_star(leaves):
    _check(leaves + 1, {(0, k) for k in range(1, leaves + 1)}, 73)


def test_star_keeps_its_time():
    from paper_2512_22215_amd import LduMatrix
    leaves = 1000
    a = _matrix(leaves + 1, {(0, k) for k in range(1, leaves + 1)}, 75)
    m = LduMatrix(leaves + 1, *map(_t, a))
    b = _t(np.random.default_rng(76).standard_normal(leaves + 1))
    m.gamg_setup(smoother="gs2")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    m.vcycle(b, **CYCLES[0])
    torch.cuda.synchronize()
    assert time.perf_counter() - t0 <= 0.25
    m.close()
