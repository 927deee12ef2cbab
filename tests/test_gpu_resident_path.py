"""Which path a solve takes, and the ways off the resident one: both paths give
the same bits, so only the solver's own report tells them apart.  A launch that
is told from the host not to start ends normally, and the launch-per-step
kernels go on from it."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, gpu_solve, host
from paper_1410_4054_amd import fk, problems as P

pytestmark = pytest.mark.gpu

CUS = 256  # compute units of an MI355X: the most workgroups of a launch
METHODS = ["cg_pipelined", "cg_pipelined_1k", "bicgstab_pipelined", "bicgstab_pipelined_2k"]


def _oracle(A, b, method, **kw):
    base = "bicgstab_pipelined" if method.startswith("bicgstab") else "cg_pipelined"
    return oracle.solve(A, b, method=base, **kw)


def _solver(A, method, layout=None, **kw):
    M = fk.Matrix(A, layout=layout)
    return fk.Solver(M, method=method, **kw)


def _shape(n):
    """Workgroups and rows: whole slices, at least 256 rows, all units."""
    slices = -(-n // 64)
    rows = max(-(-slices // CUS) * 64, 256)
    return -(-n // rows), rows


def _long(method):
    """A system that the method is still working on after 8192 iterations: the
    1D Laplacian for CG, an indefinite shifted 2D one for BiCGStab."""
    if method.startswith("cg"):
        n, i = 4500, np.arange(4500)
        return P._from_coo(n, np.concatenate([i, i[1:], i[:-1]]), np.concatenate([i, i[1:] - 1, i[:-1] + 1]),
                           np.concatenate([np.full(n, 2.0), np.full(2 * n - 2, -1.0)]))
    A = P.poisson2d(47)
    diag = A.col_idx == np.repeat(np.arange(A.n, dtype=np.int32), np.diff(A.row_ptr))
    return P.Csr(A.n, A.row_ptr, A.col_idx, A.vals - 0.3 * diag)


def _same(S, bd, ref, x0=None):
    x = dev(np.zeros(S.A.n) if x0 is None else x0)
    st = S.solve(bd, x)
    assert fk.STATUS_NAMES[st] == ref.status and S.iterations() == ref.k
    assert np.array_equal(host(x), ref.x, equal_nan=True)
    assert np.array_equal(S.history(), ref.hist[: len(S.history())], equal_nan=True)


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("nx,ny", [(4097, 1), (257, 16), (128, 128), (256, 256), (301, 218), (364, 361), (513, 512),
                                   (725, 723), (1024, 1024)])
def test_shapes_2d_are_resident(nx, ny, method, device):
    A = P.heat2d(nx, ny=ny)
    print(f"\n[case] {method} n={A.n}", flush=True)
    S = _solver(A, method, rtol=0.0, max_iter=2)
    S.solve(dev(P.rhs_uniform(A.n, 11)), dev(np.zeros(A.n)))
    assert S.resident() == (*_shape(A.n), 1, False)


@pytest.mark.parametrize("A,method", [
    (lambda: P.poisson3d(25), "cg_pipelined"), (lambda: P.poisson3d(64), "bicgstab_pipelined"),
    (lambda: P.poisson3d(80), "cg_pipelined"), (lambda: P.poisson3d(100), "cg_pipelined"),
    (lambda: P.poisson3d(128), "cg_pipelined"), (lambda: P.heat2d(1025, ny=1024), "cg_pipelined"),
    (lambda: P.heat2d(777, ny=2001), "cg_pipelined"), (lambda: P.convdiff2d(1024), "bicgstab_pipelined_2k")],
    ids=["25^3", "64^3", "80^3", "100^3", "128^3", "1025x1024", "777x2001", "cd1024"])
def test_shapes_large_are_resident(A, method, device):
    A = A()
    S = _solver(A, method, rtol=0.0, max_iter=2)
    S.solve(dev(P.rhs_uniform(A.n, 11)), dev(np.zeros(A.n)))
    assert S.resident() == (*_shape(A.n), 1, False)


@pytest.mark.parametrize("layout", ["sliced", "sliced16", "slots"])
def test_layouts_are_resident(layout, device):
    A = P.heat2d(71, ny=83)
    S = _solver(A, "cg_pipelined", layout=layout, rtol=0.0, max_iter=2)
    S.solve(dev(P.rhs_uniform(A.n, 11)), dev(np.zeros(A.n)))
    assert S.resident() == (*_shape(A.n), 1, False)


def test_one_workgroup_is_resident(device):
    for nx, ny, method in ((16, 16, "cg_pipelined"), (45, 45, "bicgstab_pipelined"), (64, 64, "cg_pipelined")):
        A = P.heat2d(nx, ny=ny)
        S = _solver(A, method, rtol=0.0, max_iter=1)
        S.solve(dev(P.rhs_uniform(A.n, 11)), dev(np.zeros(A.n)))
        assert S.uses_small() and S.resident()[0] == 1 and S.resident()[2:] == (1, False)


def test_other_paths_are_not(device):
    """What the header keeps to the launch-per-step kernels."""
    A = P.heat2d(100)
    b, x = dev(P.rhs_uniform(A.n, 11)), dev(np.zeros(A.n))
    for kw in ({"graph": True}, {"profile": True}):
        S = _solver(A, "cg_pipelined", rtol=0.0, max_iter=2, **kw)
        S.solve(b, x)
        assert S.resident() == (0, 0, 0, False), kw
    for layout, method in (("row_blocks", "cg_pipelined"), (None, "cg_classical"), (None, "cg_mixed"),
                           (None, "gmres_pipelined")):
        S = _solver(A, method, layout=layout, max_iter=2)
        S.solve(b, x)
        assert S.resident() == (0, 0, 0, False), (layout, method)
        with pytest.raises(fk.FkError) as e:
            S.test_resident(decline=1)
        assert e.value.status == fk.E_STATE


@pytest.mark.parametrize("method", METHODS)
@pytest.mark.parametrize("A", [lambda: P.convdiff2d(70), lambda: P.heat2d(257, ny=255)], ids=["70^2", "257x255"])
def test_declined_start(A, method, device):
    """The first launch does not start: the launch-per-step kernels solve from
    x0, to the tolerance and to a budget, and the next launch that is not
    declined is whole."""
    A = A()
    b = P.rhs_uniform(A.n, 5)
    x0 = np.random.default_rng(3).uniform(-1, 1, A.n)
    bd = dev(b)
    for kw in ({"rtol": 1e-8}, {"rtol": 0.0, "max_iter": 7}):
        if method.startswith("cg") and A.n == 4900 and "max_iter" not in kw:
            continue  # (CG does not converge on the nonsymmetric matrix)
        ref = _oracle(A, b, method, x0=x0, **kw)
        print(f"\n[case] declined {method} n={A.n} {kw} k={ref.k}", flush=True)
        S = _solver(A, method, **kw)
        S.test_resident(decline=1)
        _same(S, bd, ref, x0=x0)
        assert S.resident() == (*_shape(A.n), 0, True)
        S2 = _solver(A, method, **kw)
        _same(S2, bd, ref, x0=x0)
        assert S2.resident() == (*_shape(A.n), 1, False)


@pytest.mark.parametrize("method", METHODS)
def test_continuation(method, device):
    """More iterations than one launch takes: in two launches, and where the
    second does not start.  x, r, p, A p and the scalars that the first one
    (8192 iterations) left are where the next launch and the launch-per-step
    kernels of each schedule read them.  (Against those kernels from the first
    iteration on: after thousands of iterations at the rounding level of a
    stagnating solve, the oracle's exact sums are no reference any more.)"""
    A = _long(method)
    bd = dev(P.rhs_uniform(A.n, 11))
    xr = dev(np.zeros(A.n))
    R = _solver(A, method, rtol=0.0, max_iter=8195, profile=True)
    assert R.solve(bd, xr) == fk.NOT_CONVERGED and R.iterations() == 8195 and R.resident()[2] == 0
    for decline in (0, 1, 2):
        print(f"\n[case] continuation {method} declined={decline}", flush=True)
        S = _solver(A, method, rtol=0.0, max_iter=8195)
        S.test_resident(decline=decline)
        x = dev(np.zeros(A.n))
        assert S.solve(bd, x) == fk.NOT_CONVERGED and S.iterations() == 8195
        assert S.resident()[2:] == [(2, False), (0, True), (1, True)][decline]
        assert np.array_equal(host(x), host(xr))
        assert np.array_equal(S.history(), R.history())


def test_scalars_after_declined_continuation(device):
    """The per-iteration scalars across the change of path."""
    A = _long("cg_pipelined")
    b = dev(P.rhs_uniform(A.n, 11))
    out = []
    for decline in (0, 2):
        S = _solver(A, "cg_pipelined", rtol=0.0, max_iter=8200, record_history=9000, record_scalars=True)
        S.test_resident(decline=decline)
        S.solve(b, dev(np.zeros(A.n)))
        assert S.resident()[2:] == ((2, False) if decline == 0 else (1, True))
        out.append((S.history(), S.scalars()))
    assert len(out[0][0]) == len(out[1][0]) > 8192
    assert np.array_equal(out[0][0], out[1][0], equal_nan=True)
    a, b = out[0][1], out[1][1]  # alpha, beta, (omega: BiCGStab's), <r,r>
    assert len(a) == len(b) > 8192
    assert np.array_equal(a[:, 3], b[:, 3]) and np.array_equal(a[:-1, :2], b[:-1, :2])


@pytest.mark.parametrize("method", METHODS)
def test_tags_start_again(method, device):
    """The 32-bit tags run out: between two solves, with a launch declined under
    the number that now comes again, and between two launches of a solve."""
    A = P.heat2d(100)
    b = P.rhs_uniform(A.n, 5)
    bd = dev(b)
    ref = _oracle(A, b, method, rtol=1e-8)
    S = _solver(A, method)
    S.test_resident(decline=1)  # the solver's first launch: number 1
    _same(S, bd, ref)
    assert S.resident()[2:] == (0, True)
    for last in (2**32 - 1, 2**32 - 16392, 2**32 - 16393):  # the last two: one launch short of it, and just enough
        print(f"\n[case] tags {method} from {last}", flush=True)
        S = S if last == 2**32 - 1 else _solver(A, method)
        S.test_resident(next_tag=last)
        for _ in range(3):
            _same(S, bd, ref)
            assert S.resident()[2:] == (1, False)
    A = _long(method)
    bd = dev(P.rhs_uniform(A.n, 11))
    out = []
    for tag in (1, 2**32 - 1 - 16392):
        S = _solver(A, method, rtol=0.0, max_iter=8195)
        S.test_resident(next_tag=tag)
        x = dev(np.zeros(A.n))
        S.solve(bd, x)
        assert S.resident()[2:] == (2, False)
        out.append((host(x), S.history()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_declined_starts_are_remembered(device):
    """After a declined start a solver leaves the path for 1, 2, 4, ... 64 solves
    before it tries again; a launch that starts ends that."""
    A = P.heat2d(100)
    b = P.rhs_uniform(A.n, 5)
    bd = dev(b)
    ref = _oracle(A, b, "cg_pipelined", rtol=1e-8)
    S = _solver(A, "cg_pipelined")

    def solve():
        _same(S, bd, ref)
        return S.resident()[2:]

    S.test_resident(decline=1)
    for rest in (1, 2, 4, 8, 16, 32, 64, 64):
        print(f"\n[case] declined, then {rest} solves without", flush=True)
        assert solve() == (0, True)
        assert [solve() for _ in range(rest)] == [(0, False)] * rest
    S.test_resident(decline=0)
    assert solve() == (1, False) and solve() == (1, False)
    S.test_resident(decline=1)
    assert solve() == (0, True) and solve() == (0, False) and solve() == (0, True)
