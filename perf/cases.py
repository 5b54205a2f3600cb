"""Performance cases of the GPLHR library: what a program that uses it calls.

Each case is a dict of plain values.  ``prepare`` makes on the GPU what such a
program holds before the call (operands, CSR arrays, the solver handle it steps),
``run`` is one pass through the public entry points, ``exact`` the same result
from plain torch in 64 bits, ``work`` the bytes and operations of a pass.

Sizes follow the repository's named workloads: the 32^2 and 64^3 .. 160^3
convection-diffusion grids (block 4, 10, 16, trial bases of 16, 40, 64 columns)
and the diagonally dominant random pencils (17 entries per row, block 10).
"""
import math

import torch

from paper_1506_06829_amd import gplhr as G

DT = {"c128": torch.complex128, "c64": torch.complex64}
SIZE = {"c128": 16, "c64": 8}
VELOCITY = (20.0, 10.0, 5.0)
OMEGA = 0.7


def listed():
    return [
        # C X of the largest grid in the complex64 phase: the sparse product
        # that every block of the trial basis takes once or more per iteration
        dict(name="spmm 160^3 c64 x16", kind="spmm", pattern="grid", size=160, b=16, dtype="c64"),
        # the same product on an unstructured pencil, complex128, block of 10
        dict(name="spmm random c128 x10", kind="spmm", pattern="random", size=262144, b=10, dtype="c128"),
        # the damped-Jacobi preconditioner as a call of its own, 64^3 grid
        dict(name="jacobi 64^3 c128 x10", kind="jacobi", pattern="grid", size=64, b=10, dtype="c128", sweeps=3),
        # the projected pencil's Gram of the largest grid: 64 trial columns
        dict(name="gram 4096000 c64 64x64", kind="gram", n=4096000, bx=64, by=64, dtype="c64", one=False),
        # the same of a 64^3 grid or a 262144-row pencil: 40 trial columns
        dict(name="gram 262144 c128 40x40", kind="gram", n=262144, bx=40, by=40, dtype="c128", one=False),
        # the smallest workload (32^2 grid, 16 trial columns): launches count
        dict(name="gram 1024 c128 16x16", kind="gram", n=1024, bx=16, by=16, dtype="c128", one=False),
        # new V and P from the 64-column trial basis
        dict(name="update 4096000 c128 64-32", kind="update", n=4096000, wx=64, wy=32, dtype="c128", beta=0.0),
        # projection of a 5-wide block (deflation in steps of 5) against 20
        # columns, rows and widths off every tile
        dict(name="update 1000003 c64 20-5", kind="update", n=1000003, wx=20, wy=5, dtype="c64", beta=1.0),
        # the test basis of the largest grid: 48 columns against Q's 16
        dict(name="orth 4096000 c64 16+48", kind="orth", n=4096000, wy=16, w=48, dtype="c64"),
        # one iteration of the largest grid in the complex64 phase of a
        # mixed-precision handle (the whole hot path)
        dict(name="iterate 160^3 mixed x16", kind="iterate", size=160, b=16, precision="mixed"),
        # a complete FP64 solve: create, iterate to 1e-10, read the Schur form
        # (its vectors are fixed up to phases and the tolerance, so the
        # eigenvalues are what a pass returns)
        dict(name="solve 262144 fp64 k10", kind="solve", n=262144, k=10, precision="fp64"),
        # forward and backward of the eigenvalues on a small pencil
        dict(name="gradient 1024 k4", kind="gradient", n=1024, k=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("spmm", "spmm", "jacobi", "gram", "gram", "update", "update", "orth", "orth", "iterate",
                       "solve", "gradient"))
    dtype = rng.choice(("c128", "c64"))
    if kind in ("spmm", "jacobi"):
        pattern = rng.choice(("grid", "random"))
        size = _log(rng, 12, 150) if pattern == "grid" else _log(rng, 1000, 500000)
        c = dict(kind=kind, pattern=pattern, size=size, b=rng.choice((1, 4, 5, 8, 10, 12, 16, 32)), dtype=dtype)
        if kind == "jacobi":
            c["sweeps"] = rng.choice((1, 2, 3, 4))
        return c
    if kind == "gram":
        one = rng.random() < 0.4
        bx = rng.randint(1, 64)
        return dict(kind=kind, n=_log(rng, 300, 2000000), bx=bx, by=bx if one else rng.randint(1, 64), dtype=dtype,
                    one=one)
    if kind == "update":
        return dict(kind=kind, n=_log(rng, 300, 2000000), wx=rng.randint(1, 64), wy=rng.randint(1, 48), dtype=dtype,
                    beta=rng.choice((0.0, 1.0)))
    if kind == "orth":
        b = rng.choice((4, 5, 8, 10, 12, 16))
        wy, w = rng.choice(((0, 1), (1, 1), (2, 1), (3, 1), (1, 3)))
        return dict(kind=kind, n=_log(rng, 1000, 2000000), wy=wy * b, w=w * b, dtype=dtype)
    if kind == "iterate":
        return dict(kind=kind, size=rng.randint(48, 144), b=rng.choice((8, 10, 12, 16)),
                    precision=rng.choice(("mixed", "fp64")))
    if kind == "solve":
        return dict(kind=kind, n=_log(rng, 3000, 260000), k=rng.randint(4, 10), precision=rng.choice(("mixed", "fp64")))
    return dict(kind=kind, n=_log(rng, 600, 6000), k=rng.randint(2, 6))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(shape, dtype, g):
    return torch.randn(shape, dtype=dtype, device="cuda", generator=g)


def _grid(N):
    """3-D upwind convection-diffusion operator (7 points, x fastest), CSR."""
    n = N ** 3
    i = torch.arange(n, device="cuda")
    xyz = (i % N, (i // N) % N, i // (N * N))
    h = 1.0 / (N + 1)
    lap = 1.0 / h ** 2
    steps, values, inside = [], [], []
    for ax in (2, 1, 0):
        steps.append(-N ** ax)
        values.append(-lap - VELOCITY[ax] / h)
        inside.append(xyz[ax] > 0)
    steps.append(0)
    values.append(6.0 * lap + sum(VELOCITY) / h)
    inside.append(torch.ones_like(i, dtype=torch.bool))
    for ax in (0, 1, 2):
        steps.append(N ** ax)
        values.append(-lap)
        inside.append(xyz[ax] < N - 1)
    keep = torch.stack(inside, 1)
    cols = i[:, None] + torch.tensor(steps, device="cuda")[None, :]
    vals = torch.tensor(values, dtype=torch.complex128, device="cuda")[None, :].expand(n, 7)
    return _csr(n, keep.sum(1), cols[keep], vals[keep])


def _csr(n, counts, cols, vals):
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(counts, 0).to(torch.int32)
    return G.DeviceCsr(n, rp, cols.to(torch.int32).contiguous(), vals.contiguous())


def _dominant(n, g):
    """Diagonally dominant random operator: diagonal U[0, n) + 0.1 i N(0, 1),
    16 off-diagonal columns per row, one from each sixteenth of the others,
    entries 0.25 CN(0, 1) (with a block a little wider than the wanted pairs,
    every seed converges)."""
    q = 16
    r = torch.arange(n, device="cuda")
    w = (n - 1) // q
    off = 1 + w * torch.arange(q, device="cuda") + torch.randint(0, w, (n, q), device="cuda", generator=g)
    cols = torch.cat([(r[:, None] + off) % n, r[:, None]], 1)
    d = torch.complex(n * torch.rand(n, dtype=torch.float64, device="cuda", generator=g),
                      0.1 * torch.randn(n, dtype=torch.float64, device="cuda", generator=g))
    vals = torch.cat([0.25 * _randn((n, q), torch.complex128, g), d[:, None]], 1)
    cols, at = torch.sort(cols, 1)
    return _csr(n, torch.full((n,), q + 1, device="cuda"), cols.reshape(-1), torch.gather(vals, 1, at).reshape(-1))


def _diag(d):
    n = d.numel()
    return G.DeviceCsr(n, torch.arange(n + 1, dtype=torch.int32, device="cuda"),
                       torch.arange(n, dtype=torch.int32, device="cuda"), d.to(torch.complex128))


def _b_diag(n, g):
    return 1.0 + torch.rand(n, dtype=torch.float64, device="cuda", generator=g)


def _rows(A):
    return torch.repeat_interleave(torch.arange(A.n, device="cuda"), (A.row_ptr[1:] - A.row_ptr[:-1]).long())


def _shifted(A, sigma, bd):
    """C = A - sigma diag(bd); every row of A stores its diagonal."""
    r = _rows(A)
    on = A.col_idx.long() == r
    val = A.val.clone()
    val[on] -= sigma * bd
    return G.DeviceCsr(A.n, A.row_ptr, A.col_idx, val)


def _operator(case, g):
    if case["pattern"] == "grid":
        A = _grid(case["size"])
        sigma = 1000.0 + 100.0j if case["size"] > 100 else 500.0 + 50.0j
    else:
        A = _dominant(case["size"], g)
        sigma = A.n / 2 + 0.3j
    return _shifted(A, sigma, _b_diag(A.n, g))


def _inputs(case, seed):
    """The arrays of a case (the same for prepare and exact)."""
    g = _gen(seed)
    kind = case["kind"]
    if kind in ("spmm", "jacobi"):
        C = _operator(case, g)
        return C, _randn((C.n, case["b"]), DT[case["dtype"]], g)
    if kind == "gram":
        X = _randn((case["n"], case["bx"]), DT[case["dtype"]], g)
        return X, X if case["one"] else _randn((case["n"], case["by"]), DT[case["dtype"]], g)
    if kind == "update":
        X = _randn((case["n"], case["wx"]), DT[case["dtype"]], g)
        M = _randn((case["wx"], case["wy"]), torch.complex128, g) / math.sqrt(case["wx"])
        return X, M, _randn((case["n"], case["wy"]), DT[case["dtype"]], g)
    if kind == "orth":
        Z = _randn((case["n"], case["wy"] + case["w"]), DT[case["dtype"]], g)
        if case["wy"]:
            Y = Z[:, :case["wy"]].to(torch.complex128)
            for _ in range(2):
                Y = _cholqr(Y)
            Z[:, :case["wy"]] = Y.to(Z.dtype)
        return Z
    if kind in ("solve", "gradient"):
        A = _dominant(case["n"], g)
        return A, _diag(_b_diag(case["n"], g)), case["n"] / 2 + 0.3j
    A = _grid(case["size"])
    return A, _diag(_b_diag(A.n, g)), (1000.0 + 100.0j if case["size"] > 100 else 500.0 + 50.0j)


def _mul_h(X, Y):
    """X^H Y in 64 bits."""
    return X.conj().T.contiguous() @ Y


def _cholqr(X):
    R = torch.linalg.cholesky(_mul_h(X, X)).conj().T.contiguous()
    return X @ torch.linalg.inv(R)


def prepare(case, seed):
    kind = case["kind"]
    got = _inputs(case, seed)
    s = dict(kind=kind, case=case)
    if kind == "spmm":
        C, X = got
        s.update(C=C, X=X, val=C.val.to(X.dtype), plane=G.csr_plane(C), Y=torch.empty_like(X))
    elif kind == "jacobi":
        C, R = got
        s.update(C=C, R=R, plane=G.csr_plane(C))
    elif kind == "gram":
        s.update(X=got[0], Y=got[1])
    elif kind == "update":
        s.update(X=got[0], M=got[1], Y=got[2])
    elif kind == "orth":
        s.update(Z=got)
    elif kind == "iterate":
        A, B, sigma = got
        # a handle that stays in its first precision phase and is stepped
        s.update(solver=G.Solver(A, B, sigma, case["b"], case["b"], precond="jacobi", sweeps=3, omega=OMEGA,
                                 precision=case["precision"], tol=0.0, seed=seed + 1, switch_tol=0.0,
                                 stall_window=10 ** 6))
    else:
        s.update(A=got[0], B=got[1], sigma=got[2])
        if kind == "gradient":
            s.update(valA=got[0].val.clone().requires_grad_(True), valB=got[1].val.clone().requires_grad_(True))
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "spmm":
        return G.spmm(s["C"], s["X"], s["Y"], val=s["val"], plane=s["plane"])
    if kind == "jacobi":
        return G.jacobi(s["C"], s["R"], omega=OMEGA, sweeps=case["sweeps"], plane=s["plane"])
    if kind == "gram":
        return G.gram(s["X"], s["Y"])
    if kind == "update":
        return G.block_update(s["X"], s["M"], s["Y"], beta=case["beta"])
    if kind == "orth":
        return G.proj_orth(s["Z"], case["wy"], case["w"])
    if kind == "iterate":
        h = s["solver"]
        h.iterate(1)
        out = h.schur(want_vectors=False)
        lam, rho, res = out["lam"], out["rho"], h.residual_norms()
        if case["precision"] == "mixed":   # iterates of the complex64 phase carry single precision
            lam, rho, res = lam.astype("c8"), rho.astype("f4"), res.astype("f4")
        return dict(lam=lam, rho=rho, residual=res)
    block = case["k"] + 4
    if kind == "solve":
        h = G.Solver(s["A"], s["B"], s["sigma"], case["k"], block, precond="diag", precision=case["precision"],
                     tol=1e-10, max_iter=200, seed=7)
        h.iterate()
        out = h.schur()
        h.close()
        return out["lam"]
    s["valA"].grad = s["valB"].grad = None
    lam = G.GPLHREig.apply(s["valA"], s["valB"], s["A"], s["B"], s["sigma"], case["k"],
                           dict(block=block, precond="diag", tol=1e-13, max_iter=200))
    (lam - s["sigma"]).abs().square().sum().backward()
    return dict(lam=lam.detach(), gradA=s["valA"].grad, gradB=s["valB"].grad)


# --------------------------------------------------------------------------
# bytes and operations
# --------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("spmm", "jacobi"):
        n = case["size"] ** 3 if case["pattern"] == "grid" else case["size"]
        nnz = 7 * n - 6 * case["size"] ** 2 if case["pattern"] == "grid" else 17 * n
        e, b = SIZE[case["dtype"]], case["b"]
        if kind == "spmm":
            return dict(bytes=nnz * (e + 4) + 4 * (n + 1) + 2 * n * b * e, flops=8 * nnz * b)
        return dict(bytes=nnz * 20 + 4 * (n + 1) + 2 * n * b * e, flops=8 * max(1, case["sweeps"] - 1) * nnz * b)
    if kind == "gram":
        w = case["bx"] + (0 if case["one"] else case["by"])
        pairs = case["bx"] * (case["bx"] + 1) // 2 if case["one"] else case["bx"] * case["by"]
        return dict(bytes=case["n"] * w * SIZE[case["dtype"]] + 16 * case["bx"] * case["by"], flops=8 * case["n"] * pairs)
    if kind == "update":
        read = case["wx"] + (case["wy"] if case["beta"] else 0)
        return dict(bytes=case["n"] * (read + case["wy"]) * SIZE[case["dtype"]], flops=8 * case["n"] * case["wx"] * case["wy"])
    if kind == "orth":
        n, wy, w = case["n"], case["wy"], case["w"]
        # two passes: coefficients against Y, the block's own Gram, the update
        return dict(bytes=n * (wy + 2 * w) * SIZE[case["dtype"]], flops=2 * 8 * n * (2 * wy * w + w * (w + 1)))
    if kind == "iterate":
        n, b = case["size"] ** 3, case["b"]
        nnz = 7 * n - 6 * case["size"] ** 2
        s, e = 4 * b, 8 if case["precision"] == "mixed" else 16
        # V, C V, Q and P in and out once, the operator once; seven sparse
        # products and the projected pencil's two Grams and four basis updates
        return dict(bytes=8 * n * b * e + nnz * (e + 4) + 20 * n, flops=56 * nnz * b + 8 * n * (2 * s * s + 5 * s * b))
    n, k = case["n"], case["k"]
    return dict(bytes=17 * n * 20 + 16 * n * (2 * k + 1), flops=4 * 8 * 17 * n * k * (2 if kind == "gradient" else 1))


# --------------------------------------------------------------------------
# 64-bit results
# --------------------------------------------------------------------------
def _apply(C, rows, val, X):
    """C X in 64 bits, a few columns at a time."""
    Y = torch.zeros((C.n, X.shape[1]), dtype=torch.complex128, device="cuda")
    col = C.col_idx.long()
    for c in range(0, X.shape[1], 4):
        part = val[:, None] * X[:, c:c + 4][col]
        out = torch.zeros((C.n, part.shape[1], 2), dtype=torch.float64, device="cuda")
        out.index_add_(0, rows, torch.view_as_real(part))
        Y[:, c:c + 4] = torch.view_as_complex(out)
    return Y


def exact(case, seed):
    kind = case["kind"]
    if kind in ("iterate", "solve") or (kind == "gradient" and case["n"] > 1100):
        return None
    got = _inputs(case, seed)
    if kind == "spmm":
        C, X = got
        return _apply(C, _rows(C), C.val.to(X.dtype).to(torch.complex128), X.to(torch.complex128))
    if kind == "jacobi":
        C, R = got
        R, rows = R.to(torch.complex128), _rows(C)
        dw = (OMEGA / C.val[C.col_idx.long() == rows])[:, None]
        w = dw * R
        for _ in range(case["sweeps"] - 1):
            w = w + dw * (R - _apply(C, rows, C.val, w))
        return w
    if kind == "gram":
        return _mul_h(got[0].to(torch.complex128), got[1].to(torch.complex128))
    if kind == "update":
        X, M, Y = got
        return case["beta"] * Y.to(torch.complex128) + X.to(torch.complex128) @ M
    if kind == "orth":
        Z, wy = got.to(torch.complex128), case["wy"]
        Y, X = Z[:, :wy].contiguous(), Z[:, wy:].contiguous()
        for _ in range(2):
            if wy:
                X = X - Y @ _mul_h(Y, X)
            X = _cholqr(X)
        Z[:, wy:] = X
        return Z
    # dense eigenvalues and eigenvectors of B^{-1} A; left vectors from the inverse
    A, B, sigma = got
    n, k = A.n, case["k"]
    rows, cols = _rows(A).cpu(), A.col_idx.long().cpu()
    D = torch.zeros((n, n), dtype=torch.complex128)
    D[rows, cols] = A.val.cpu()
    bd = B.val.cpu()
    lam, X = torch.linalg.eig(D / bd[:, None])
    at = torch.argsort((lam - sigma).abs())[:k]
    Yh = torch.linalg.inv(X)[at] / bd[None, :]         # y^H with y^H B x = 1
    lam, X = lam[at], X[:, at]
    coef = 2 * (lam - sigma)
    # dL/dA_ij = sum_e coef_e conj(y^H_i x_j), B alike with -conj(lambda)
    gA = (coef[None, :] * (Yh.conj().T[rows] * X.conj()[cols])).sum(1)
    i = torch.arange(n)
    gB = -(coef[None, :] * lam.conj()[None, :] * (Yh.conj().T[i] * X.conj()[i])).sum(1)
    return dict(lam=lam, gradA=gA, gradB=gB)
