"""Timed cases of the library's public entry points, each a thing that a
program built on it does: one product, one solve, one step of a transient
run, one batch, one training gradient.

  listed()            the cases that stand for the range
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what the program holds before the call
  run(state)          one pass, and its outputs
  work(case)          bytes and operations a pass cannot do without
  exact(case, seed)   the same outputs from plain numpy / torch in 64 bits

Matrices are the generators of paper_1410_4054_amd.problems; right-hand
sides, vectors and fields come from the seed.  Solves start from x = 0 and
run to the relative residual named in the case.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1410_4054_amd import fk
from paper_1410_4054_amd import problems as P

DEV = "cuda"
HEAT_C = 4.0   # dt kappa / h^2 of the heat operator I + c L5
SHIFT = 0.25   # diagonal shift of an implicit convection-diffusion step


def listed():
    return [
        # A small irregular matrix (empty rows, a few long ones: the row-block
        # layout), one product with its two inner products: the smallest call.
        {"name": "spmv_irregular_20k", "kind": "spmv", "n": 20011, "nnz": 4, "empty": 200, "long": 4},
        # The random-column matrix of the fused product benchmark, 28 per row.
        {"name": "spmv_random28_1m", "kind": "spmv", "n": 1000000, "nnz": 28, "empty": 0, "long": 0},
        # Latency-bound systems: a thousand unknowns, one workgroup's work.
        {"name": "cg_poisson2d_32", "kind": "cg2d", "n": 32, "method": "cg_pipelined", "rtol": 1e-8},
        # Small-to-medium 2D system: launches and reductions, not bandwidth.
        {"name": "cg_poisson2d_127", "kind": "cg2d", "n": 127, "method": "cg_pipelined", "rtol": 1e-8},
        # The benchmark's workload: 3D Poisson, 2.1 M unknowns.
        {"name": "cg_poisson3d_128", "kind": "cg3d", "n": 128, "method": "cg_pipelined", "rtol": 1e-8},
        # Beyond the 256 MB cache: 7.1 M unknowns.
        {"name": "cg_poisson3d_192", "kind": "cg3d", "n": 192, "method": "cg_pipelined", "rtol": 1e-8},
        # The nonsymmetric benchmark, BiCGStab in two kernels per iteration.
        {"name": "bicgstab_convdiff_1024", "kind": "bicgstab", "n": 1024, "method": "bicgstab_pipelined_2k",
         "rtol": 1e-8},
        # One implicit step of convection-diffusion with GMRES(30).
        {"name": "gmres30_convdiff_1024", "kind": "gmres", "n": 1024, "method": "gmres_pipelined",
         "restart": 30, "rtol": 1e-8},
        # FP32 inner iterations in FP64 refinement.
        {"name": "mixed_f32_poisson3d_128", "kind": "mixed", "n": 128, "method": "cg_mixed_f32", "rtol": 1e-10},
        # Many uneven systems in one launch.
        {"name": "batch_128_uneven", "kind": "batch", "count": 128, "nmin": 16, "nmax": 512, "rtol": 1e-10},
        # One time step of the heat equation: right-hand side, learned guess, solve.
        {"name": "heat_step_512", "kind": "heat", "n": 512, "method": "cg_pipelined_1k", "layers": 4,
         "passes": 4, "rtol": 1e-8},
        # One training sample: features, forward, loss, backward.
        {"name": "net_gradient_512", "kind": "gradient", "n": 512, "layers": 4, "act": "linear"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["spmv", "cg2d", "cg3d", "bicgstab", "gmres", "mixed", "batch", "heat", "gradient"])
    if kind == "spmv":
        irregular = rng.random() < 0.4
        n = _log_int(rng, 5000 if irregular else 1000, 1000000)
        return {"kind": kind, "n": n, "nnz": rng.randint(4, 28 if n < 500000 else 12),
                "empty": n // 100 if irregular else 0, "long": rng.randint(1, 8) if irregular else 0}
    if kind == "cg2d":
        return {"kind": kind, "n": _log_int(rng, 15, 800), "method": rng.choice(["cg_pipelined", "cg_pipelined_1k"]),
                "rtol": 1e-8}
    if kind == "cg3d":
        return {"kind": kind, "n": _log_int(rng, 10, 150), "method": "cg_pipelined", "rtol": 1e-8}
    if kind == "bicgstab":
        return {"kind": kind, "n": _log_int(rng, 15, 700),
                "method": rng.choice(["bicgstab_pipelined", "bicgstab_pipelined_2k"]), "rtol": 1e-8}
    if kind == "gmres":
        return {"kind": kind, "n": _log_int(rng, 31, 1024), "method": "gmres_pipelined",
                "restart": rng.choice([20, 30]), "rtol": 1e-8}
    if kind == "mixed":
        return {"kind": kind, "n": _log_int(rng, 16, 128), "method": rng.choice(["cg_mixed_f32", "cg_mixed"]),
                "rtol": 1e-10}
    if kind == "batch":
        nmax = _log_int(rng, 64, 400)
        return {"kind": kind, "count": rng.randint(16, 128), "nmin": 16, "nmax": nmax, "rtol": 1e-10}
    if kind == "heat":
        return {"kind": kind, "n": _log_int(rng, 64, 640), "method": rng.choice(["cg_pipelined", "cg_pipelined_1k"]),
                "layers": rng.randint(2, 5), "passes": rng.randint(1, 4), "rtol": 1e-8}
    return {"kind": kind, "n": _log_int(rng, 64, 640), "layers": rng.randint(2, 6),
            "act": rng.choice(["linear", "relu"])}


# ------------------------------------------------------------------ inputs

@functools.lru_cache(maxsize=2)
def _matrix(kind: str, n: int, nnz: int = 0, empty: int = 0, long: int = 0):
    """Host CSR of a case; the assembly is not part of any pass."""
    if kind == "spmv":
        step = max(1, n // max(1, long))
        rows = {i * step + step // 2: min(3000, n) for i in range(long)}
        return P.random_csr(n, nnz, seed=0, empty_rows=empty, long_rows=rows)
    if kind == "cg2d":
        return P.poisson2d(n)
    if kind in ("cg3d", "mixed"):
        return P.poisson3d(n)
    if kind == "bicgstab":
        return P.convdiff2d(n)
    a = P.convdiff2d(n)
    on_diag = a.col_idx == np.repeat(np.arange(a.n, dtype=np.int32), np.diff(a.row_ptr))
    return P.Csr(a.n, a.row_ptr, a.col_idx, a.vals + SHIFT * on_diag)


def _case_matrix(case):
    return _matrix(case["kind"], case["n"], case.get("nnz", 0), case.get("empty", 0), case.get("long", 0))


def _rhs(n: int, seed: int):
    return np.random.default_rng(seed).uniform(-1.0, 1.0, n)


def _heat_fields(n: int, seed: int):
    """A, u_{m-1}, u_m, dt f^m and dt f^{m+1} of the second step (m = 1) of a
    transient run: u_m solves A u_m = u_{m-1} + dt f^m."""
    A, u0, source = P.heat_transient(n, seed + 1, 400)
    f1, f2 = source(1), source(2)
    line = (n, -HEAT_C, 0.0, -HEAT_C)
    u1 = _separable_solve([(n, -HEAT_C, 1.0 + 4.0 * HEAT_C, -HEAT_C), line], u0 + f1)
    return A, u0, u1, f2


@functools.lru_cache(maxsize=2)
def _batch_pattern(count: int, nmin: int, nmax: int):
    """The batch's sizes and block-diagonal matrix, with where its diagonal lies."""
    A, sys_ptr, _ = P.batch_problem(count, 0, nmin, nmax)
    diag = np.flatnonzero(A.col_idx == np.repeat(np.arange(A.n, dtype=np.int32), np.diff(A.row_ptr)))
    return A, sys_ptr, diag


def _batch(case, seed):
    """(A, sys_ptr, shift, b): the sizes are the case's, the diagonal shifts
    in [0, 0.1) and the right-hand sides the seed's."""
    A, sys_ptr, diag = _batch_pattern(case["count"], case["nmin"], case["nmax"])
    rng = np.random.default_rng(seed)
    shift = rng.uniform(0.0, 0.1, A.n)
    vals = A.vals.copy()
    vals[diag] = 4.0 + shift
    return P.Csr(A.n, A.row_ptr, A.col_idx, vals), sys_ptr, shift, rng.uniform(-1.0, 1.0, A.n)


def _dev(a):
    return torch.as_tensor(a, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "spmv":
        A = _case_matrix(case)
        return {"case": case, "M": fk.Matrix(A), "p": _dev(_rhs(A.n, seed)),
                "q": torch.zeros(A.n, dtype=torch.float64, device=DEV)}
    if kind == "batch":
        A, sys_ptr, _, b = _batch(case, seed)
        return {"case": case, "B": fk.Batch(A, sys_ptr), "b": _dev(b),
                "x": torch.zeros(A.n, dtype=torch.float64, device=DEV)}
    if kind in ("heat", "gradient"):
        A, u0, u1, f2 = _heat_fields(case["n"], seed)
        net = fk.Net(case["layers"], P.net_init(case["layers"], seed), activation=case.get("act", "linear"))
        st = {"case": case, "M": fk.Matrix(A), "net": net, "um1": _dev(u0), "um": _dev(u1)}
        if kind == "heat":
            st.update(f=_dev(f2), b=torch.empty(A.n, dtype=torch.float64, device=DEV),
                      x=torch.empty(A.n, dtype=torch.float64, device=DEV))
            st["S"] = fk.Solver(st["M"], method=case["method"], rtol=case["rtol"], record_history=False,
                                unroll=4, small=False)
        else:
            line = (case["n"], -HEAT_C, 0.0, -HEAT_C)
            b = u1 + f2
            unext = _separable_solve([(case["n"], -HEAT_C, 1.0 + 4.0 * HEAT_C, -HEAT_C), line], b)
            st.update(b=_dev(b), unext=_dev(unext))
        return st
    A = _case_matrix(case)
    M = fk.Matrix(A)
    S = fk.Solver(M, method=case["method"], rtol=case["rtol"], record_history=False,
                  restart=case.get("restart", 0))
    return {"case": case, "M": M, "S": S, "b": _dev(_rhs(A.n, seed)),
            "x": torch.zeros(A.n, dtype=torch.float64, device=DEV)}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "spmv":
        pq, qq = fk.spmv(st["M"], st["p"], st["q"], dots=True)
        return {"q": st["q"], "pq": pq, "qq": qq}
    if kind == "batch":
        st["x"].zero_()
        st["B"].solve(st["b"], st["x"], rtol=case["rtol"])
        r = st["B"].results()
        return {"x": st["x"], "status": r.status, "iterations": r.iterations, "sweeps": r.sweeps}
    if kind == "heat":
        n = case["n"]
        fk.axpby(1.0, st["um"], 1.0, st["f"], st["b"])
        st["net"].guess(st["M"], n, n, st["b"], st["um"], st["um1"], st["x"], passes=case["passes"])
        status = st["S"].solve(st["b"], st["x"])
        return {"b": st["b"], "x": st["x"], "status": status}
    if kind == "gradient":
        n = case["n"]
        grad, loss = st["net"].gradient(st["M"], n, n, st["b"], st["um"], st["um1"], st["unext"])
        return {"grad": grad, "loss": loss}
    st["x"].zero_()
    status = st["S"].solve(st["b"], st["x"])
    return {"x": st["x"], "status": status, "iterations": st["S"].iterations()}


# -------------------------------------------------------------------- work

def _iterations(case):
    """About how many products a solve takes (measured at a few sizes)."""
    kind, n = case["kind"], case["n"]
    if kind == "cg2d":
        return 3.0 * (n + 1)
    if kind == "cg3d":
        return 3.45 * (n + 1)
    if kind == "bicgstab":
        return 2 * 1.9 * (n + 1)
    if kind == "mixed":
        return 6.5 * (n + 1)
    return 60.0


def work(case):
    """Every product of a solve reads the matrix values and a vector and
    writes a vector, once each (FP32 where the method's inner iterations are
    FP32); 2 operations per nonzero and 10 per unknown for the updates and
    inner products.  GMRES also reads its basis (half of `restart` vectors on
    average) for the inner products."""
    kind = case["kind"]
    if kind == "spmv":
        n = case["n"]
        nnz = (n - case["empty"]) * case["nnz"] + case["long"] * min(3000, n)
        return {"bytes": 12.0 * nnz + 20.0 * n, "flops": 2.0 * nnz + 4.0 * n}
    if kind == "batch":
        lo, hi, c = case["nmin"], case["nmax"], case["count"]
        # E[n^2] and E[n^3] of a uniform side; about 4 (n+1) FP32 iterations each
        n2 = (hi ** 3 - lo ** 3) / (3.0 * (hi - lo))
        n3 = (hi ** 4 - lo ** 4) / (4.0 * (hi - lo))
        its_rows = c * min(4.0 * n3, 250.0 * n2)
        return {"bytes": its_rows * (5 * 4 + 8) + c * n2 * 16, "flops": its_rows * 20.0}
    if kind in ("heat", "gradient"):
        N = float(case["n"]) ** 2
        nnz = 5 * N - 4 * case["n"]
        hidden = case["layers"] - 2
        conv = 2.0 * 9 * N * (16 + 16 * 16 * hidden + 16)
        if kind == "heat":
            its = 10.0
            return {"bytes": case["passes"] * (12 * nnz + 40 * N) + its * (8 * nnz + 16 * N) + 24 * N,
                    "flops": case["passes"] * conv + its * (2 * nnz + 10 * N)}
        # features; each hidden activation written once and read once backward
        return {"bytes": 12 * nnz + 40 * N + (case["layers"] - 1) * 2 * 32 * N, "flops": 3 * conv}
    dim = 3 if kind in ("cg3d", "mixed") else 2
    N = float(case["n"]) ** dim
    nnz = (2 * dim + 1) * N - 2 * dim * N / case["n"]
    its = _iterations(case)
    word = 4 if kind == "mixed" else 8
    per = word * nnz + 2 * word * N
    if kind == "gmres":
        per += 0.5 * case["restart"] * 8 * N
    return {"bytes": its * per, "flops": its * (2 * nnz + 10 * N)}


# ----------------------------------------------------- the same in 64 bits

def _sines(n):
    k = np.arange(1, n + 1)
    return np.sqrt(2.0 / (n + 1)) * np.sin(np.outer(k, k) * (np.pi / (n + 1)))


def _separable_solve(lines, b):
    """Solve (T_x + T_y [+ T_z]) x = b for tridiagonal Toeplitz lines
    (n, lower, diagonal, upper), x first and fastest: sine transforms in
    every direction but x, elimination along x."""
    shape = [ln[0] for ln in lines][::-1]
    v = np.asarray(b, dtype=np.float64).reshape(shape)
    lam = np.zeros(shape[:-1])
    undo = []
    for d, (n, lo, di, up) in enumerate(lines[1:], start=1):
        ax = len(lines) - 1 - d
        S = _sines(n)
        scale = np.sqrt(lo / up) ** np.arange(n)
        cut = [1] * len(shape)
        cut[ax] = n
        v = np.moveaxis(np.tensordot(S, v / scale.reshape(cut), axes=(1, ax)), 0, ax)
        e = di + 2.0 * np.copysign(np.sqrt(lo * up), up) * np.cos(np.arange(1, n + 1) * np.pi / (n + 1))
        lam = lam + e.reshape(cut[:-1])
        undo.append((ax, S, scale.reshape(cut)))
    n, lo, di, up = lines[0]
    v = np.ascontiguousarray(np.moveaxis(v, -1, 0))
    diag = lam + di
    c = np.empty_like(v)
    c[0] = up / diag
    v[0] = v[0] / diag
    for i in range(1, n):
        den = diag - lo * c[i - 1]
        c[i] = up / den
        v[i] = (v[i] - lo * v[i - 1]) / den
    for i in range(n - 2, -1, -1):
        v[i] -= c[i] * v[i + 1]
    v = np.moveaxis(v, 0, -1)
    for ax, S, scale in reversed(undo):
        v = np.moveaxis(np.tensordot(S, v, axes=(1, ax)), 0, ax) * scale
    return np.ascontiguousarray(v).ravel()


def _case_lines(case):
    n, kind = case["n"], case["kind"]
    if kind == "cg2d":
        return [(n, -1.0, 4.0, -1.0), (n, -1.0, 0.0, -1.0)]
    if kind in ("cg3d", "mixed"):
        return [(n, -1.0, 6.0, -1.0), (n, -1.0, 0.0, -1.0), (n, -1.0, 0.0, -1.0)]
    h = 1.0 / (n + 1)
    vx, vy = 50.0, 25.0
    d = 4.0 + h * (vx + vy) + (SHIFT if kind == "gmres" else 0.0)
    return [(n, -(1.0 + h * vx), d, -1.0), (n, -(1.0 + h * vy), 0.0, -1.0)]


def _exact_batch(case, seed):
    """Per system (L5 + diag(shift)) x = b: sine-transform solves with the
    mean shift as the preconditioner, repeated until the correction vanishes."""
    out = []
    _, sys_ptr, shifts, rhs = _batch(case, seed)
    for r0, r1 in zip(sys_ptr[:-1], sys_ptr[1:]):
        ns, shift, b = math.isqrt(int(r1 - r0)), shifts[r0:r1], rhs[r0:r1]
        S = torch.as_tensor(_sines(ns), device=DEV)
        e = 2.0 - 2.0 * torch.cos(torch.arange(1, ns + 1, device=DEV, dtype=torch.float64) * (math.pi / (ns + 1)))
        inv = 1.0 / (e[:, None] + e[None, :] + 0.05)
        d = 4.0 + _dev(shift).reshape(ns, ns)
        bb = _dev(b).reshape(ns, ns)
        x = torch.zeros_like(bb)
        for _ in range(60):
            r = bb - d * x
            r[1:] += x[:-1]
            r[:-1] += x[1:]
            r[:, 1:] += x[:, :-1]
            r[:, :-1] += x[:, 1:]
            x = x + S @ ((S @ r @ S) * inv) @ S
        out.append(x.reshape(-1).cpu().numpy())
    return np.concatenate(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "spmv":
        A = _case_matrix(case)
        p = _rhs(A.n, seed)
        rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
        q = np.bincount(rows, weights=A.vals * p[A.col_idx], minlength=A.n)
        return {"q": q, "pq": math.fsum(p * q), "qq": math.fsum(q * q)}
    if kind == "batch":
        return {"x": _exact_batch(case, seed), "status": None, "iterations": None, "sweeps": None}
    if kind in ("heat", "gradient"):
        n = case["n"]
        A, u0, u1, f2 = _heat_fields(n, seed)
        line = (n, -HEAT_C, 0.0, -HEAT_C)
        b = u1 + f2
        x = _separable_solve([(n, -HEAT_C, 1.0 + 4.0 * HEAT_C, -HEAT_C), line], b)
        if kind == "heat":
            return {"b": b, "x": x, "status": None}
        g = 2.0 * u1 - u0
        rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
        r = b - np.bincount(rows, weights=A.vals * g[A.col_idx], minlength=A.n)
        s = float(np.max(np.abs(r)))
        plane = torch.as_tensor(r / s).reshape(1, 1, n, n)
        target = torch.as_tensor((x - g) / s).reshape(1, 1, n, n)
        w = torch.as_tensor(P.net_init(case["layers"], seed)).double().requires_grad_(True)
        off, a = 0, plane
        for layer in range(case["layers"]):
            ci = 1 if layer == 0 else 16
            co = 1 if layer == case["layers"] - 1 else 16
            a = torch.nn.functional.conv2d(a, w[off: off + co * ci * 9].reshape(co, ci, 3, 3), padding=1)
            off += co * ci * 9
            if case["act"] == "relu" and layer < case["layers"] - 1:
                a = torch.relu(a)
        loss = torch.mean((a - target) ** 2)
        loss.backward()
        return {"grad": w.grad.numpy(), "loss": float(loss.detach())}
    return {"x": _separable_solve(_case_lines(case), _rhs(case["n"] ** (3 if kind in ("cg3d", "mixed") else 2), seed)),
            "status": None, "iterations": None}
