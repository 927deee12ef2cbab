"""The resident solver (a whole solve in one launch of workgroups that own
their rows) against the oracle, bit for bit, where its shapes change: the
last workgroup's remainder, rows per thread 1 to 16 at both thread
counts, one workgroup, one and two hand-overs per reduction, 5 and 7 entries per row, every
sliced layout, ghosts on both sides and more of them than the threads hold
at once.  Solves run a fixed number of iterations (rtol 0) or to 1e-8."""
import threading

import numpy as np
import pytest

import oracle
from gpu_util import dev, gpu_solve, host
from paper_1410_4054_amd import fk, problems as P

pytestmark = pytest.mark.gpu


def _check(A, its, layout=None, method="cg_pipelined", x0=None):
    b = P.rhs_uniform(A.n, 11)
    base = "bicgstab_pipelined" if method.startswith("bicgstab") else "cg_pipelined"
    ref = oracle.solve(A, b, x0=x0, method=base, rtol=0.0, max_iter=its)
    res, x = gpu_solve(A, b, x0, method=method, rtol=0.0, max_iter=its, layout=layout)
    print(f"[case] n={A.n} {method} {layout} k={res.k}", flush=True)
    assert (res.status, res.k) == (ref.status, ref.k)
    assert np.array_equal(x, ref.x)
    assert np.array_equal(res.history, ref.hist[: len(res.history)])


# n one more and one less than whole workgroups (256 rows up to n = 65,536,
# then n / 256), at the steps of rows per thread (256, 512, 1024, 2048, 4096
# rows) and at 64 workgroups (16,384), where the hand-over changes
@pytest.mark.parametrize("method", ["cg_pipelined", "bicgstab_pipelined_2k"])
@pytest.mark.parametrize("nx,ny", [(4097, 1), (257, 16), (128, 128), (5, 3277), (256, 256), (301, 218), (364, 361),
                                   (512, 512), (513, 512), (725, 723), (1024, 1024)])
def test_rows_2d(nx, ny, method, device):
    _check(P.heat2d(nx, ny=ny), 5, method=method)


@pytest.mark.parametrize("method", ["cg_pipelined", "bicgstab_pipelined"])
@pytest.mark.parametrize("n", [17, 25, 41, 64, 65, 80])
def test_rows_3d(n, method, device):
    _check(P.poisson3d(n), 4, method=method)


# the matrix streamed (more than 4096 rows per workgroup, or more ghosts than
# fit beside 4096), bricks that do not divide the grid
@pytest.mark.parametrize("A", [lambda: P.heat2d(1025, ny=1024), lambda: P.heat2d(777, ny=2001),
                               lambda: P.poisson3d(100), lambda: P.poisson3d(103)],
                         ids=["1025x1024", "777x2001", "100^3", "103^3"])
def test_streamed(A, device):
    _check(A(), 4)


# one workgroup: rows per thread 1, 2, 2, 4, 8, whole and partial slices
@pytest.mark.parametrize("nx,ny", [(1, 1), (15, 17), (16, 16), (257, 1), (32, 32), (45, 45), (41, 50), (64, 64)])
def test_rows_one_workgroup(nx, ny, device):
    its = min(6, nx * ny)
    _check(P.heat2d(nx, ny=ny), its)
    if nx * ny <= 2048:
        _check(P.heat2d(nx, ny=ny), its, method="bicgstab_pipelined_2k")


# sizes past the single workgroup's (2048 for BiCGStab, 3072 for the one-kernel
# CG) and below and at 16 whole workgroups
@pytest.mark.parametrize("nx,ny", [(683, 3), (439, 7), (63, 65), (64, 64)])
def test_rows_few_workgroups(nx, ny, device):
    _check(P.heat2d(nx, ny=ny), 6, method="bicgstab_pipelined_2k")
    _check(P.heat2d(nx, ny=ny), 6, method="cg_pipelined_1k")


@pytest.mark.parametrize("n", [7, 12, 16])
def test_rows_one_workgroup_3d(n, device):
    _check(P.poisson3d(n), 6)


@pytest.mark.parametrize("method", ["cg_pipelined_1k", "bicgstab_pipelined_2k"])
@pytest.mark.parametrize("layout", ["sliced", "sliced16", "slots"])
def test_layouts(layout, method, device):
    x0 = np.random.default_rng(2).uniform(-1, 1, 71 * 83)
    _check(P.heat2d(71, ny=83), 9, layout=layout, method=method, x0=x0)


@pytest.mark.parametrize("method", ["bicgstab_pipelined", "bicgstab_pipelined_2k"])
def test_bicgstab_decisions(method, device):
    """Every end of a BiCGStab solve: the tolerance on the expanded norm, the
    half step, the budget after each of the first iterations, b = 0."""
    A = P.convdiff2d(70)
    b = P.rhs_uniform(A.n, 5)
    for rtol, its in ((1e-8, None), (1e-3, None), (0.0, 1), (0.0, 2), (0.0, 3)):
        ref = oracle.solve(A, b, method="bicgstab_pipelined", rtol=rtol, max_iter=its)
        res, x = gpu_solve(A, b, method=method, rtol=rtol, max_iter=its)
        assert (res.status, res.k) == (ref.status, ref.k) and np.array_equal(x, ref.x), (rtol, its)
        assert np.array_equal(res.history, ref.hist)
    I4 = P.scaled_identity(5000, 4.0)  # s_0 = 0: the half step ends the solve
    b = P.rhs_uniform(5000, 6)
    res, x = gpu_solve(I4, b, method=method)
    assert (res.status, res.k) == ("converged", 1) and np.array_equal(x, b / 4.0)
    res, x = gpu_solve(I4, np.zeros(5000), np.ones(5000), method=method)
    assert (res.status, res.k) == ("converged", 0) and not x.any()


def test_scattered_columns(device):
    """Rows of unequal length with columns anywhere: ghosts in many pieces,
    duplicated columns, rows without entries, more ghosts than threads."""
    rng = np.random.default_rng(4)
    n = 9000
    counts = rng.integers(0, 4, n)
    rows = np.repeat(np.arange(n), counts)
    cols = rng.integers(0, n, rows.size)
    vals = rng.uniform(-0.1, 0.1, rows.size)
    i = np.arange(n)
    A = P._from_coo(n, np.concatenate([i, rows, cols]), np.concatenate([i, cols, rows]),
                    np.concatenate([np.full(n, 2.0), vals, vals]))
    if np.diff(A.row_ptr).max() > 7:  # keep the widest row within the kernels' seven
        keep = np.arange(A.nnz) - np.repeat(A.row_ptr[:-1], np.diff(A.row_ptr)) < 7
        cnt = np.minimum(np.diff(A.row_ptr), 7)
        A = P.Csr(n, np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32), A.col_idx[keep], A.vals[keep])
    _check(A, 6, layout="sliced")


def test_long_solve_continues(device):
    """More iterations than one launch takes (8192): r, p and A p come back
    from memory, by the parity of the count, and the run is the oracle's."""
    A = P.heat2d(70, ny=64)
    for method in ("cg_pipelined", "cg_pipelined_1k"):
        _check(A, 8195, method=method)
    A = P.convdiff2d(65)
    for method in ("bicgstab_pipelined", "bicgstab_pipelined_2k"):
        b = P.rhs_uniform(A.n, 11)
        ref = oracle.solve(A, b, method="bicgstab_pipelined", rtol=0.0, max_iter=8194)
        res, x = gpu_solve(A, b, method=method, rtol=0.0, max_iter=8194)
        assert (res.status, res.k) == (ref.status, ref.k) and np.array_equal(x, ref.x, equal_nan=True)


def test_concurrent_streams(device):
    """Four threads, each with a stream and a solver of its own: together they
    want more compute units than there are, so some take the other path."""
    import torch

    A = P.heat2d(400, ny=300)
    b = P.rhs_uniform(A.n, 1)
    ref, xref = gpu_solve(A, b)
    M = fk.Matrix(A)
    out = [None] * 4

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
            bd = dev(b)
            S = fk.Solver(M, stream=s)
            got = []
            for _ in range(5):
                x.zero_()
                st = S.solve(bd, x)
                got.append((st, S.iterations(), host(x)))
            S.close()
        out[t] = got

    ts = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for got in out:
        for st, k, x in got:
            assert st == fk.OK and k == ref.k and np.array_equal(x, xref)
