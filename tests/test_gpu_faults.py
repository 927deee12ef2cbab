"""Waits that run out: a reduction of which one leader gives up is void, and
the call says so.  The condition is asked for from the host; every kernel ends
normally."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host
from paper_1410_4054_amd import fk, problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["slots", "row_blocks"])
@pytest.mark.parametrize("n,groups", [(512, (0, 3)), (40, (0,))], ids=["groups", "one-group"])
def test_spmv_leader_gives_up(n, groups, layout, device):
    """A leader below the top one hands an incomplete sum on that the top
    leader takes for a whole one; the call must not.  The next call on the
    matrix is whole."""
    A = P.poisson2d(n)
    p = np.random.default_rng(1).uniform(-1, 1, A.n)
    M = fk.Matrix(A, layout=layout)
    pd, qd = dev(p), dev(np.zeros(A.n))
    want = fk.spmv(M, pd, qd, dots=True)
    assert np.array_equal(host(qd), oracle.spmv(A, p))
    for group in groups:
        print(f"\n[case] spmv {layout} n={A.n}: leader of group {group} gives up", flush=True)
        M.test_fault(group)
        with pytest.raises(fk.FkError, match="did not complete") as e:
            fk.spmv(M, pd, qd, dots=True)
        assert e.value.status == fk.E_HIP
        assert fk.spmv(M, pd, qd, dots=True) == want
        M.test_fault(group)
        with pytest.raises(fk.FkError, match="did not complete"):
            fk.spmv(M, pd, qd, dots=True)
        assert fk.spmv_time(M, pd, qd, mode="fused", reps=2) > 0.0


def test_spmv_test_fault_arguments(device):
    M = fk.Matrix(P.poisson2d(8))
    for group in (-1, 64):
        with pytest.raises(fk.FkError) as e:
            M.test_fault(group)
        assert e.value.status == fk.E_ARG


def test_spmv_dots_of_many_matrices(device):
    """The pinned words that the dots arrive in are shared out among the
    matrices, 64 to a page: three pages in use, given back in another order and
    taken again."""
    rng = np.random.default_rng(2)
    mats = [P.poisson2d(4 + i % 7) for i in range(150)]
    ps = [rng.uniform(-1, 1, A.n) for A in mats]
    want = []
    for A, p in zip(mats, ps):
        q = oracle.spmv(A, p)
        want.append((float(p @ q), float(q @ q)))
    Ms = [fk.Matrix(A) for A in mats]

    def check(i):
        got = fk.spmv(Ms[i], dev(ps[i]), dev(np.zeros(mats[i].n)), dots=True)
        # (numpy's sums of at most 100 products: within 100 roundings)
        assert np.allclose(got, want[i], rtol=0, atol=100 * 2.0 ** -53 * 8 * mats[i].n), i

    for i in range(150):
        check(i)
    for i in rng.permutation(150)[:120]:
        Ms[i].close()
        Ms[i] = None
    for i in range(150):
        if Ms[i] is None:
            Ms[i] = fk.Matrix(mats[i])
    for i in rng.permutation(150):
        check(int(i))
