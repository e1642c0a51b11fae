"""Calls that run out of device memory part way, and the same call again: every array that
a first solve asks for is refused once (ldu_deny_memory), the call returns LDU_ERR_NOMEM,
and the call after it gives what an undisturbed handle gives, bit for bit.  An operator,
vector set or FP32 copy of which only a part was made must not count as there.

The hierarchies are built for the Gauss-Seidel smoother, which needs none of the operators
of the Jacobi cycles, so that the cycles make theirs themselves.
"""
import numpy as np
import pytest

from meshgen import box_case, random_order, relabel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GENERAL = dict(n_pre=2, n_post=2)
ONE_SWEEP = dict(n_pre=1, n_post=1, scale_correction=0)


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _deny(m, n):
    from paper_2512_22215_amd import ldu as LL
    return LL.lib().ldu_deny_memory(m.handle, n)


def _again(m, call, fresh=None, denied=None):
    """call(m) with the n-th array refused, then call(m) as it is, for n = 1, 2, ...
    (or those in `denied`): the number of calls that failed.  fresh(): a handle to use."""
    from paper_2512_22215_amd.ldu import LDU_ERR_NOMEM, LduError
    h = fresh() if fresh else m
    _deny(h, 0)
    ref = call(h)
    count = _deny(h, 0)
    failed = 0
    for n in denied or range(1, count + 1):
        h = fresh() if fresh else m
        _deny(h, n)
        with pytest.raises(LduError) as err:
            call(h)
        assert err.value.code == LDU_ERR_NOMEM, n
        failed += 1
        assert torch.equal(call(h), ref), n
    return failed


@pytest.mark.parametrize("cycle", [GENERAL, ONE_SWEEP], ids=["general", "one-sweep"])
@pytest.mark.parametrize("mixed", [False, True])
def test_operators_of_a_cycle(cycle, mixed):
    from paper_2512_22215_amd import LduMatrix
    c = box_case(9, 8, 7, coeff="lognormal", dirichlet_x0=1.0, seed=5)
    b = _t(c.rhs[0])

    def fresh():
        m = LduMatrix.from_case(c)
        m.gamg_setup(smoother="gs2")
        return m

    def call(m):
        if not mixed:
            return m.vcycle(b, **cycle)
        return m.gamg(b, precision="mixed", rel_tol=0.0, max_refine=2, **cycle)[0]
    assert _again(None, call, fresh) > 20


def test_operators_of_a_large_plain_level():
    from paper_2512_22215_amd import LduMatrix
    c = box_case(90, 90, 90, coeff="lognormal", dirichlet_x0=1.0, seed=6)
    m = LduMatrix.from_case(c)
    b = _t(c.rhs[0])

    def fresh():
        m.gamg_setup(smoother="gs2")
        return m
    fresh()
    m.vcycle(b, **ONE_SWEEP)
    assert m.downleg(0) == ("scaled_slices", 0)
    # the two value arrays, the mapped columns, their bases and the flag, then a
    # CSR level's first arrays
    assert _again(None, lambda h: h.vcycle(b, **ONE_SWEEP), fresh, range(1, 9)) == 8
    # calls that fail after the large arrays are made do not keep them
    from paper_2512_22215_amd.ldu import LduError
    fresh()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(20):
        _deny(m, 5)
        with pytest.raises(LduError):
            m.vcycle(b, **ONE_SWEEP)
    assert torch.cuda.mem_get_info()[0] >= free - 8 * c.n_cells
    m.close()


@pytest.mark.parametrize("solver", ["pcg", "pbicg"])
def test_vectors_of_a_first_solve(solver):
    from paper_2512_22215_amd import LduMatrix
    c = box_case(9, 8, 7, coeff="lognormal", dirichlet_x0=1.0, nonsym=0.3, seed=7)
    b = _t(c.rhs[0])

    def call(m):
        return getattr(m, solver)(b, rel_tol=0.0, max_iter=5)[0]
    assert _again(None, call, lambda: LduMatrix.from_case(c)) >= 2


def test_setup_and_renewed_setup():
    from paper_2512_22215_amd import LduMatrix
    c = box_case(9, 8, 7, coeff="lognormal", dirichlet_x0=1.0, seed=8)
    m = LduMatrix.from_case(c)
    b = _t(c.rhs[0])

    def call(h):
        h.gamg_setup(**ONE_SWEEP)
        return h.vcycle(b, **ONE_SWEEP)
    call(m)
    assert _again(m, call) > 100
    m.close()


def test_scattered_mesh_without_memory_for_renumbered_levels():
    """The copies of the levels are a gain in speed: without memory for them the solves run
    on the levels as they are."""
    from paper_2512_22215_amd import LduMatrix
    c = box_case(80, 80, 80, coeff="lognormal", dirichlet_x0=1.0, seed=9)
    c = relabel(c, random_order(c.n_cells, np.random.default_rng(10)))
    m = LduMatrix.from_case(c)
    b = _t(c.rhs[0])
    _deny(m, 0)
    m.gamg_setup(smoother="gs2")
    levels = _deny(m, 0) - 4 * m.n_levels() - 2  # without the work vectors
    plain = m.vcycle(b, **GENERAL)
    m.gamg_setup(**GENERAL)
    assert not torch.equal(m.vcycle(b, **GENERAL), plain)  # another order of sums
    for k in (2, 7, 40, 90):  # 1: the test of the numbering
        _deny(m, levels + k)
        m.gamg_setup(**GENERAL)
        assert torch.equal(m.vcycle(b, **GENERAL), plain), k
    m.gamg_setup(**GENERAL)
    assert not torch.equal(m.vcycle(b, **GENERAL), plain)
    m.close()
