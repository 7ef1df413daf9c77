"""Timed cases of the solver: the calls that a program makes on the way from a
dense or bidiagonal matrix to its singular value decomposition, each through
the public binding (``paper_2508_11467_amd.api.Solver``).

Families (``kind``):
  svd      one bidiagonal solve, ``Solver.svd``: sigma, U, V^T
  batch    many bidiagonals of uneven sizes in one ``Solver.svd_batched`` call
  qr       Householder QR of a tall matrix and its explicit Q
           (``geqrf`` + ``orgqr``)
  gebrd    reduction of a dense matrix to bidiagonal form
  backtr   a bidiagonal reduction's reflectors applied to the singular vectors
  gemm     the plain FP64 product that ends a tall-and-skinny SVD (U = Q U_R)

A program keeps one handle for its life, so the handles are shared by every
state of a process.  Inputs are new tensors for every state.  A call that
overwrites its argument gets a copy of the state's input, as a program makes
that still needs the original.
"""

import math

import numpy as np
import torch

from paper_2508_11467_amd import inputs
from paper_2508_11467_amd.api import Solver

F64 = torch.float64
_HANDLES = {}


def _handle(gemm="fp64"):
    """The program's handle with this arithmetic of the update products."""
    if gemm not in _HANDLES:
        _HANDLES[gemm] = Solver(0, gemm=gemm)
    return _HANDLES[gemm]


def listed():
    return [
        # the smallest call: latency of one small bidiagonal
        {"name": "svd_n100_uniform", "kind": "svd", "n": 100, "spectrum": "uniform", "gemm": "fp64", "out": False},
        # the bidiagonal of a tall-and-skinny SVD's R factor
        {"name": "svd_n1000_normal", "kind": "svd", "n": 1000, "spectrum": "normal", "gemm": "fp64", "out": False},
        # mid size, values over eight decades
        {"name": "svd_n4096_graded", "kind": "svd", "n": 4096, "spectrum": "graded", "gemm": "fp64", "out": False},
        # the headline size, results into buffers that the program keeps
        {"name": "svd_n16384_normal", "kind": "svd", "n": 16384, "spectrum": "normal", "gemm": "fp64", "out": True},
        # hardly any deflation: bound by the vector-update products
        {"name": "svd_n6000_near_ones", "kind": "svd", "n": 6000, "spectrum": "near_ones", "gemm": "fp64", "out": True},
        # the same with the split-precision products
        {"name": "svd_n6000_near_ones_crt", "kind": "svd", "n": 6000, "spectrum": "near_ones", "gemm": "crt",
         "out": True},
        # many small and mid-size problems in one call
        {"name": "batch2000_32_2048", "kind": "batch", "count": 2000, "lo": 32, "hi": 2048},
        # first and fifth step of the SVD of a tall matrix
        {"name": "qr_20000x1000", "kind": "qr", "m": 20000, "n": 1000},
        # dense square SVD: the reduction
        {"name": "gebrd_4096", "kind": "gebrd", "m": 4096, "n": 4096},
        # dense square SVD: U = Q U_2 (column-stored reflectors)
        {"name": "backtr_8192_cols", "kind": "backtr", "m": 8192, "p": 8192, "rows": False},
        # dense SVD of an odd size: V = P V_2 (row-stored reflectors)
        {"name": "backtr_3001_rows", "kind": "backtr", "m": 3001, "p": 3001, "rows": True},
        # last step of the SVD of a tall matrix
        {"name": "gemm_20000x1000x1000", "kind": "gemm", "m": 20000, "n": 1000, "k": 1000},
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; every third one a
    multiple of 64, as sizes in programs often are."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    x = round(x / 64) * 64 if rng.random() < 0.34 else round(x)
    return int(min(hi, max(lo, x)))


def draw(rng):
    kind = rng.choice(["svd", "svd", "svd", "batch", "qr", "gebrd", "backtr", "gemm"])
    if kind == "svd":
        spectrum = rng.choice(["normal", "uniform", "graded", "clustered", "near_ones"])
        if spectrum == "near_ones":
            return {"kind": "svd", "n": _log_int(rng, 300, 6000), "spectrum": spectrum,
                    "gemm": rng.choice(["fp64", "crt"]), "out": rng.random() < 0.5}
        return {"kind": "svd", "n": _log_int(rng, 32, 16384), "spectrum": spectrum, "gemm": "fp64",
                "out": rng.random() < 0.5}
    if kind == "batch":
        return {"kind": "batch", "count": _log_int(rng, 10, 2000), "lo": 32, "hi": _log_int(rng, 64, 2048)}
    if kind == "qr":
        n = _log_int(rng, 20, 1000)
        return {"kind": "qr", "m": _log_int(rng, max(n, 300), 20000), "n": n}
    if kind == "gebrd":
        n = _log_int(rng, 64, 2000)
        return {"kind": "gebrd", "m": _log_int(rng, n, 2 * n), "n": n}
    if kind == "backtr":
        m = _log_int(rng, 200, 8192)
        return {"kind": "backtr", "m": m, "p": _log_int(rng, 64, m), "rows": rng.random() < 0.5}
    return {"kind": "gemm", "m": _log_int(rng, 300, 20000), "n": _log_int(rng, 32, 1000), "k": _log_int(rng, 32, 1000)}


# ------------------------------------------------------------------ inputs
def _dense(rows, cols, seed):
    """A rows x cols N(0, 1) matrix on the device, column-major."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((cols, rows), dtype=F64, device="cuda", generator=g).T


def _empty(rows, cols):
    return torch.empty((cols, rows), dtype=F64, device="cuda").T


def _bidiagonal(case, seed):
    n, s = case["n"], case["spectrum"]
    make = {"normal": inputs.normal, "uniform": inputs.uniform, "graded": inputs.graded,
            "clustered": inputs.clustered, "near_ones": inputs.near_ones}[s]
    return make(n, seed)


def _batch(case, seed):
    # the sizes are the workload, the entries the input
    sizes = inputs.batch_sizes(case["count"], case["lo"], case["hi"], 2508)
    return sizes, inputs.batch_uniform(sizes, seed)


def _reflectors(case, seed):
    """Reflectors as a reduction leaves them: unit pivots at entry i (columns)
    or i + 1 (rows), the stored entries of norm just below 1, tau = 2 / y^T y.
    Returned as the (m, m) column-major matrix that a reduction overwrites,
    with the other half holding its other reflectors."""
    m = case["m"]
    A = _dense(m, m, seed)
    stored = torch.triu(A, 2) if case["rows"] else torch.tril(A, -1)
    dim = 1 if case["rows"] else 0
    norm = torch.sqrt(torch.sum(stored * stored, dim=dim, keepdim=True))
    scale = 0.97 / torch.where(norm > 0, norm, torch.ones_like(norm))
    A.mul_(scale)
    size = torch.sum((stored * scale) ** 2, dim=dim)
    tau = 2.0 / (1.0 + size)
    return A, (tau[:m - 1].contiguous() if case["rows"] else tau)


def prepare(case, seed):
    k = case["kind"]
    if k == "svd":
        d, e = _bidiagonal(case, seed)
        n = case["n"]
        out = None
        if case["out"]:
            out = tuple(torch.empty(s, dtype=F64, device="cuda") for s in ((n,), (n, n), (n, n)))
        return {"kind": k, "solver": _handle(case["gemm"]), "d": torch.from_numpy(d).cuda(),
                "e": torch.from_numpy(e).cuda(), "out": out}
    s = _handle()
    if k == "batch":
        sizes, (d, e) = _batch(case, seed)
        return {"kind": k, "solver": s, "sizes": sizes.tolist(), "d": torch.from_numpy(d).cuda(),
                "e": torch.from_numpy(e).cuda()}
    if k in ("qr", "gebrd"):
        A = _dense(case["m"], case["n"], seed)
        return {"kind": k, "solver": s, "A": A, "work": _empty(case["m"], case["n"])}
    if k == "backtr":
        Y, tau = _reflectors(case, seed)
        C = _dense(case["m"], case["p"], seed + 1) / math.sqrt(case["m"])
        return {"kind": k, "solver": s, "Y": Y, "tau": tau, "C": C, "work": _empty(case["m"], case["p"]),
                "rows": case["rows"]}
    A, B = _dense(case["m"], case["k"], seed), _dense(case["k"], case["n"], seed + 1)
    return {"kind": k, "solver": s, "A": A, "B": B, "C": _empty(case["m"], case["n"])}


# ------------------------------------------------------------------ one pass
def run(state):
    s, k = state["solver"], state["kind"]
    if k == "svd":
        sigma, U, VT = s.svd(state["d"], state["e"], out=state["out"])
        return {"sigma": sigma, "U": U, "VT": VT}
    if k == "batch":
        sigma, U, VT = s.svd_batched(state["sizes"], state["d"], state["e"])
        return {"sigma": sigma, "U": U, "VT": VT}
    if k == "qr":
        W = state["work"]
        W.copy_(state["A"])
        tau = s.geqrf(W)
        return {"A": W, "tau": tau, "Q": s.orgqr(W, tau)}
    if k == "gebrd":
        W = state["work"]
        W.copy_(state["A"])
        d, e, tauq, taup = s.gebrd(W)
        return {"A": W, "d": d, "e": e, "tauq": tauq, "taup": taup}
    if k == "backtr":
        W = state["work"]
        W.copy_(state["C"])
        s.apply_reflectors(state["Y"], state["tau"], W, offset=1 if state["rows"] else 0, rows=state["rows"])
        return {"C": W}
    s.gemm(state["A"], state["B"], state["C"])
    return {"C": state["C"]}


# ------------------------------------------------------------------ 64 bits
def _reflect(x):
    """beta, scaled entries below the pivot and tau of the reflector of x."""
    alpha, sigma = x[0].item(), torch.dot(x[1:], x[1:]).item()
    if sigma == 0.0:
        return alpha, x[1:], 0.0
    beta = -math.copysign(math.sqrt(alpha * alpha + sigma), alpha)
    den = alpha - beta
    return beta, x[1:] / den, 2.0 / (1.0 + sigma / (den * den))


def _full(y):
    return torch.cat([torch.ones(1, dtype=F64, device=y.device), y])


def _exact_qr(A):
    A = A.contiguous()
    m, n = A.shape
    tau = torch.zeros(n, dtype=F64, device=A.device)
    for c in range(n):
        beta, y, t = _reflect(A[c:, c])
        v = _full(y)
        if c + 1 < n and t:
            A[c:, c + 1:].addr_(v, v @ A[c:, c + 1:], alpha=-t)
        A[c, c] = beta
        A[c + 1:, c] = y
        tau[c] = t
    Q = torch.eye(m, n, dtype=F64, device=A.device)
    for c in range(n - 1, -1, -1):
        v = _full(A[c + 1:, c])
        Q[c:, c:].addr_(v, v @ Q[c:, c:], alpha=-tau[c].item())
    return {"A": A, "tau": tau, "Q": Q}


def _exact_gebrd(A):
    A = A.contiguous()
    m, n = A.shape
    d, e = torch.zeros(n, dtype=F64, device=A.device), torch.zeros(max(n - 1, 0), dtype=F64, device=A.device)
    tauq, taup = torch.zeros_like(d), torch.zeros_like(d)
    for c in range(n):
        beta, y, t = _reflect(A[c:, c])
        v = _full(y)
        if c + 1 < n and t:
            A[c:, c + 1:].addr_(v, v @ A[c:, c + 1:], alpha=-t)
        A[c, c] = d[c] = beta
        A[c + 1:, c] = y
        tauq[c] = t
        if c + 1 < n:
            beta, y, t = _reflect(A[c, c + 1:])
            u = _full(y)
            if t:
                A[c + 1:, c + 1:].addr_(A[c + 1:, c + 1:] @ u, u, alpha=-t)
            A[c, c + 1] = e[c] = beta
            A[c, c + 2:] = y
            taup[c] = t
    return {"A": A, "d": d, "e": e, "tauq": tauq, "taup": taup}


def _svdvals(d, e):
    return np.linalg.svd(np.diag(d) + np.diag(e[:len(d) - 1], 1), compute_uv=False)


def exact(case, seed):
    """Singular vectors have no one value in 64 bits (their signs, and their
    basis where values are close, are free), so only sigma is given for a
    solve, and only where a dense SVD on the host is quick."""
    k = case["kind"]
    if k == "svd":
        if case["n"] > 1500:
            return None
        return {"sigma": torch.from_numpy(_svdvals(*_bidiagonal(case, seed))), "U": None, "VT": None}
    if k == "batch":
        sizes, (d, e) = _batch(case, seed)
        if int(np.sum(sizes ** 3)) > 4e9 or len(sizes) > 500:
            return None
        off = np.concatenate([[0], np.cumsum(sizes)])
        got = [_svdvals(d[a:b], e[a:b]) for a, b in zip(off[:-1], off[1:])]
        return {"sigma": torch.from_numpy(np.concatenate(got)), "U": None, "VT": None}
    if k == "qr":
        return _exact_qr(_dense(case["m"], case["n"], seed))
    if k == "gebrd":
        return _exact_gebrd(_dense(case["m"], case["n"], seed))
    if k == "backtr":
        Y, tau = _reflectors(case, seed)
        C = (_dense(case["m"], case["p"], seed + 1) / math.sqrt(case["m"])).contiguous()
        for i in range(tau.shape[0] - 1, -1, -1):
            o = i + 1 if case["rows"] else i
            v = _full(Y[i, o + 1:] if case["rows"] else Y[o + 1:, i])
            C[o:].addr_(v, v @ C[o:], alpha=-tau[i].item())
        return {"C": C}
    A, B = _dense(case["m"], case["k"], seed), _dense(case["k"], case["n"], seed + 1)
    return {"C": A.contiguous() @ B.contiguous()}


# ------------------------------------------------------------------ work
def work(case):
    """Each input read once and each output written once; the operations that
    the method needs where they do not depend on the values."""
    k = case["kind"]
    if k == "svd":
        n = case["n"]
        # both sides' update products without deflation; a spectrum that
        # deflates needs next to none
        return {"bytes": 8.0 * (3 * n + 2 * n * n), "flops": 8 / 3 * n ** 3 if case["spectrum"] == "near_ones" else 0.0}
    if k == "batch":
        n = inputs.batch_sizes(case["count"], case["lo"], case["hi"], 2508).astype(float)
        return {"bytes": 8.0 * float(np.sum(3 * n + 2 * n * n)), "flops": 0.0}
    if k == "qr":
        m, n = case["m"], case["n"]
        return {"bytes": 8.0 * 3 * m * n, "flops": 2 * (2.0 * m * n * n - 2 / 3 * n ** 3)}
    if k == "gebrd":
        m, n = case["m"], case["n"]
        return {"bytes": 8.0 * 2 * m * n, "flops": 4.0 * n * n * (m - n / 3)}
    if k == "backtr":
        m, p = case["m"], case["p"]
        return {"bytes": 8.0 * (m * m / 2 + 2 * m * p), "flops": 2.0 * m * m * p}
    m, n, q = case["m"], case["n"], case["k"]
    return {"bytes": 8.0 * (m * q + q * n + m * n), "flops": 2.0 * m * n * q}
