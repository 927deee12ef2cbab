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
