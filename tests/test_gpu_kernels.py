"""Parity of the single HIP kernels (through the C ABI) with their definitions
on the CPU: sparse matrix times block, the FP64-accumulated Gram matrix and
the row-local block update."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1506_06829_amd import problems

pytestmark = pytest.mark.gpu


def _rand_csr(n, rng, max_row=40, empty_every=7):
    rows, cols = [], []
    for i in range(n):
        if i % empty_every == 3:
            continue                                  # empty rows
        m = int(rng.integers(0, max_row))             # ragged lengths
        c = np.unique(rng.integers(0, n, m))
        rows += [i] * len(c)
        cols += list(c)
    v = rng.standard_normal(len(rows)) + 1j * rng.standard_normal(len(rows))
    return problems.csr_from_scipy(sp.coo_matrix((v, (rows, cols)), shape=(n, n)))


def _block(rng, n, b, ld=None):
    ld = ld or b
    X = rng.standard_normal((n, ld)) + 1j * rng.standard_normal((n, ld))
    return X


@pytest.mark.parametrize("b", [1, 3, 4, 10, 16, 33])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_spmm_matches_definition(device, b, dtype):
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(b)
    for csr in [_rand_csr(1001, rng), problems.convection_diffusion(9, (20.0, 10.0, 5.0))]:
        n = csr.n
        A = G.DeviceCsr.from_host(csr)
        X = _block(rng, n, b, ld=b + 2)              # strided block: ld = b + 2
        tdt = torch.complex128 if dtype == "c128" else torch.complex64
        Xd = torch.as_tensor(X).to(device, tdt)[:, :b]
        Y = G.spmm(A, Xd, val=A.val.to(tdt)).cpu().numpy()
        ref = csr.to_scipy() @ X[:, :b].astype(np.complex64 if dtype == "c64" else np.complex128)
        tol = 1e-14 if dtype == "c128" else 2e-6
        scale = np.abs(csr.to_scipy()) @ np.abs(X[:, :b]) + 1e-300
        assert np.max(np.abs(Y - ref) / scale) < tol
        # bitwise reproducible
        Y2 = G.spmm(A, Xd, val=A.val.to(tdt)).cpu().numpy()
        assert np.array_equal(Y, Y2)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("b", [2, 10, 16])
def test_spmm_batch_lengths(device, dtype, b):
    # nnz only picks how many entries of a row are gathered at once (8, 12 or
    # 17 by nnz / n): every choice accumulates a row in the same order, so the
    # products are bitwise equal, and equal the definition; rows of up to 79
    # entries take several batches of each length
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(100 + b)
    csr = _rand_csr(777, rng, max_row=80, empty_every=5)
    n = csr.n
    A = G.DeviceCsr.from_host(csr)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    X = torch.as_tensor(_block(rng, n, b)).to(device, tdt)
    val = A.val.to(tdt)
    outs = []
    for hint in (0, 8 * n, 10 * n, 12 * n, 13 * n, 17 * n, 100 * n):
        Y = torch.empty_like(X)
        G._check(G.lib().gplhr_spmm(0 if dtype == "c128" else 1, n, hint, G._ptr(A.row_ptr),
                                    G._ptr(A.col_idx), G._ptr(val), G._ptr(X), b, G._ptr(Y), b, b,
                                    0, G._stream_ptr()))
        outs.append(Y.cpu().numpy())
    for Y in outs[1:]:
        assert np.array_equal(Y, outs[0])
    Xh = X.cpu().numpy()
    ref = csr.to_scipy().astype(Xh.dtype) @ Xh
    scale = np.abs(csr.to_scipy()) @ np.abs(Xh) + 1e-300
    tol = 1e-14 if dtype == "c128" else 2e-6
    assert np.max(np.abs(outs[0] - ref) / scale) < tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("sweeps", [1, 2, 3, 4])
def test_jacobi_matches_oracle(device, dtype, sweeps):
    # the preconditioner T (damped Jacobi from zero) against the oracle's, on
    # a 3-D upwind stencil (7 entries per row, plane schedule), the shifted
    # diagonally dominant pencil (17 per row) and a ragged random pattern with
    # a dominant diagonal (rows of 1..40 entries)
    import torch
    from oracle import gplhr_oracle as O
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(10 + sweeps)
    sten = problems.convection_diffusion(16, (20.0, 10.0, 5.0))
    Ad, Bd = problems.diag_dominant_pencil(3000, seed=2)
    sig = 1500.0 + 0.3j
    Cd = Ad.to_scipy() - sig * Bd.to_scipy()
    Cr = _rand_csr(999, rng).to_scipy()
    Cr = Cr + sp.diags(3.0 * np.abs(Cr).sum(axis=1).A1 + 1.0)
    for C, plane in [(sten.to_scipy(), 256), (sp.csr_matrix(Cd), 0), (sp.csr_matrix(Cr), 0)]:
        C.sort_indices()
        csr = problems.csr_from_scipy(C)
        A = G.DeviceCsr.from_host(csr)
        T = O.make_preconditioner(C, "jacobi", sweeps=sweeps, omega=0.7)
        tdt = torch.complex128 if dtype == "c128" else torch.complex64
        for b in (1, 10, 16):
            R = _block(rng, csr.n, b)
            Rd = torch.as_tensor(R).to(device, tdt)
            Y = G.jacobi(A, Rd, omega=0.7, sweeps=sweeps, plane=plane).cpu().numpy()
            ref = T(Rd.cpu().numpy().astype(np.complex128))
            tol = 1e-13 if dtype == "c128" else 5e-6
            assert np.max(np.abs(Y - ref)) < tol * np.max(np.abs(ref)), (C.shape, b)
            if plane:
                Y0 = G.jacobi(A, Rd, omega=0.7, sweeps=sweeps).cpu().numpy()
                assert np.array_equal(Y, Y0)


def test_jacobi_zero_diagonal(device):
    import torch
    from paper_1506_06829_amd import gplhr as G
    C = sp.csr_matrix(np.array([[2.0, 1.0, 0.0], [1.0, 0.0, 1.0], [0.0, 1.0, 2.0]], dtype=complex))
    A = G.DeviceCsr.from_host(problems.csr_from_scipy(C))
    R = torch.ones((3, 2), dtype=torch.complex128, device=device)
    with pytest.raises(Exception, match="zero entries"):
        G.jacobi(A, R)


def test_spmm_empty_matrix_rows(device):
    import torch
    from paper_1506_06829_amd import gplhr as G
    n = 50
    csr = problems.Csr(n, np.zeros(n + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.complex128))
    A = G.DeviceCsr.from_host(csr)
    X = torch.ones((n, 4), dtype=torch.complex128, device=device)
    Y = G.spmm(A, X).cpu().numpy()
    assert np.all(Y == 0)


@pytest.mark.parametrize("N", [16, 24])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_spmm_plane_schedule(device, N, dtype):
    # the plane-slab row order computes every row exactly as the natural order
    import torch
    from paper_1506_06829_amd import gplhr as G
    csr = problems.convection_diffusion(N, (20.0, 10.0, 5.0))
    A = G.DeviceCsr.from_host(csr)
    assert G.csr_plane(A) == (N * N if N * N >= 512 else 0)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    rng = np.random.default_rng(N)
    for b in (1, 10, 16):
        X = torch.as_tensor(_block(rng, csr.n, b)).to(device, tdt)
        Y0 = G.spmm(A, X, val=A.val.to(tdt)).cpu().numpy()
        for plane in (N * N, 8 * N, 8):
            Y1 = G.spmm(A, X, val=A.val.to(tdt), plane=plane).cpu().numpy()
            assert np.array_equal(Y0, Y1), (b, plane)


def test_csr_plane_of_unstructured_patterns(device):
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(3)
    assert G.csr_plane(G.DeviceCsr.from_host(_rand_csr(8192, rng, max_row=6))) == 0
    # 2-D stencil: the bandwidth N gives fewer than 512 rows per plane
    assert G.csr_plane(G.DeviceCsr.from_host(problems.convection_diffusion(64, (1.0, 1.0)))) == 0
    with pytest.raises(Exception, match="bad arguments"):
        A = G.DeviceCsr.from_host(problems.convection_diffusion(16, (1.0, 1.0, 1.0)))
        import torch
        X = torch.zeros((A.n, 4), dtype=torch.complex128, device=device)
        G.spmm(A, X, plane=24)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("sweeps", [1, 2, 3, 5])
def test_jacobi_zero_diagonal_leaves_output(device, dtype, sweeps):
    # the zero is found on the device: no sweep may write Y before the error
    import torch
    from paper_1506_06829_amd import gplhr as G
    C = sp.random(300, 300, density=0.02, random_state=3, format="lil").astype(complex)
    C.setdiag(4.0)
    C[77, 77] = 0.0
    A = G.DeviceCsr.from_host(problems.csr_from_scipy(sp.csr_matrix(C)))
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    R = torch.ones((300, 6), dtype=tdt, device=device)
    Y = torch.full((300, 6), 7.0, dtype=tdt, device=device)
    rc = G.lib().gplhr_jacobi(0 if dtype == "c128" else 1, A.n, A.nnz, G._ptr(A.row_ptr), G._ptr(A.col_idx),
                              G._ptr(A.val), 0.7, sweeps, G._ptr(R), 6, G._ptr(Y), 6, 6, 0, G._stream_ptr())
    assert rc == -1 and bool((Y == 7.0).all())


@pytest.mark.parametrize("b", [1, 2, 5, 16, 33, 64])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("lengths", [(5,), (7,), (0, 3, 12), (17,), (0, 0, 130, 1), (40, 300, 2)])
def test_spmm_row_lengths(device, b, dtype, lengths):
    # rows that fill a batch of gathers, fall short of it or run past it, empty
    # rows, and wavefronts whose entries do and do not fit their stage; block
    # rows that no entry refers to hold NaN.  A row of L entries sums L products:
    # (L + 2) eps of the sum of moduli.
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(b + sum(lengths))
    n = 1031
    cnt = np.array([lengths[i % len(lengths)] for i in range(n)])
    ip = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    ci = rng.integers(0, n - 7, ip[-1]).astype(np.int32)
    ci = np.concatenate([np.sort(ci[ip[i]:ip[i + 1]]) for i in range(n)]).astype(np.int32)
    val = rng.standard_normal(ip[-1]) + 1j * rng.standard_normal(ip[-1])
    X = _block(rng, n, b)
    if dtype == "c64":
        val, X = (z.astype(np.complex64).astype(np.complex128) for z in (val, X))
    A = sp.csr_matrix((val, ci, ip), shape=(n, n))
    ref = A @ X
    scale = abs(A) @ np.abs(X)
    X[n - 7:] = np.nan
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    dA = G.DeviceCsr(n, torch.as_tensor(ip).to(device), torch.as_tensor(ci).to(device),
                     torch.as_tensor(val).to(device))
    ld = b + (b % 3)
    Xd = torch.zeros((n, ld), dtype=tdt, device=device)
    Xd[:, :b] = torch.as_tensor(X).to(device, tdt)
    Y = G.spmm(dA, Xd[:, :b], val=dA.val.to(tdt)).cpu().numpy().astype(np.complex128)
    eps = 2.3e-16 if dtype == "c128" else 1.2e-7
    assert np.all(np.abs(Y - ref) <= 4 * (max(lengths) + 2) * eps * scale)


def test_spmm_of_many_tiny_planes(device):
    # planes of 8 rows: more workgroups than a launch takes, so the rows run in
    # natural order; the result is the same
    import torch
    from paper_1506_06829_amd import gplhr as G
    n = 8 * ((1 << 21) + 5)
    rp = torch.arange(n + 1, dtype=torch.int32, device=device)
    g = torch.Generator(device=device).manual_seed(2)
    v = torch.randn(n, dtype=torch.complex128, device=device, generator=g)
    A = G.DeviceCsr(n, rp, rp[:n].flip(0).contiguous(), v)
    X = torch.randn((n, 2), dtype=torch.complex128, device=device, generator=g)
    Y = G.spmm(A, X, plane=8)
    assert torch.equal(Y, G.spmm(A, X))
    ref = v[:, None] * X.flip(0)
    assert float((Y - ref).abs().max()) < 1e-14 * float(ref.abs().max())


def test_spmm_of_rows_far_apart(device):
    # a block that spans more than 32-bit byte offsets
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(4)
    n, ld, b = 40, 7_000_000, 6
    A = sp.random(n, n, density=0.3, random_state=5, format="csr") + sp.identity(n, format="csr")
    dA = G.DeviceCsr.from_host(problems.csr_from_scipy(A))
    x = _block(rng, n, b)
    X = torch.zeros((n - 1) * ld + b, dtype=torch.complex128, device=device).as_strided((n, b), (ld, 1))
    X.copy_(torch.as_tensor(x))
    Y = G.spmm(dA, X).cpu().numpy()
    assert np.all(np.abs(Y - A @ x) <= 4 * (n + 2) * 2.3e-16 * (abs(A) @ np.abs(x)))


@pytest.mark.parametrize("b", [2, 10, 16, 24, 40])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("rows", ["first", "sorted", "even", "long"])
def test_spmm_of_unevenly_spread_entries(device, b, dtype, rows):
    # most entries in the first eighth of the rows, rising row lengths (both: rows in
    # turn), even rows (by eighths), and a few rows that no stage holds among short
    # ones.  A row of L entries sums L products: (L + 2) eps of the sum of moduli.
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(b)
    n = 20011
    cnt = np.full(n, 5)
    if rows == "first":
        cnt[:n // 8] = 60
    elif rows == "sorted":
        cnt = np.sort(rng.integers(0, 30, n))
    elif rows == "long":
        cnt[::40] = 300
    ip = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    r = np.repeat(np.arange(n), cnt)
    ci = rng.integers(0, n, ip[-1])
    ci = ci[np.lexsort((ci, r))].astype(np.int32)
    val = rng.standard_normal(ip[-1]) + 1j * rng.standard_normal(ip[-1])
    X = _block(rng, n, b)
    if dtype == "c64":
        val, X = (z.astype(np.complex64).astype(np.complex128) for z in (val, X))
    A = sp.csr_matrix((val, ci, ip), shape=(n, n))
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    dA = G.DeviceCsr(n, torch.as_tensor(ip).to(device), torch.as_tensor(ci).to(device),
                     torch.as_tensor(val).to(device))
    Y = G.spmm(dA, torch.as_tensor(X).to(device, tdt), val=dA.val.to(tdt)).cpu().numpy().astype(np.complex128)
    eps = 2.3e-16 if dtype == "c128" else 1.2e-7
    scale = abs(A) @ np.abs(X)
    assert np.all(np.abs(Y - A @ X) <= 4 * (cnt.max() + 2) * eps * scale)


@pytest.mark.parametrize("plane", [64, 512, 2048])
@pytest.mark.parametrize("b", [1, 2, 5, 16])
def test_spmm_of_thin_slabs(device, plane, b):
    # planes whose slabs hold fewer rows than some workgroups take: in natural order,
    # the same bits
    import torch
    from paper_1506_06829_amd import gplhr as G
    n = 2048 * 21
    A = sp.diags([1.0, -2.0, 4.0, 0.5, 3.0], [-plane, -1, 0, 1, plane], shape=(n, n), format="csr")
    dA = G.DeviceCsr.from_host(problems.csr_from_scipy(A.astype(complex)))
    x = _block(np.random.default_rng(b), n, b)
    X = torch.as_tensor(x).to(device)
    Y = G.spmm(dA, X, plane=plane)
    assert torch.equal(Y, G.spmm(dA, X))
    assert np.max(np.abs(Y.cpu().numpy() - A @ x)) < 7 * 2.3e-16 * 11 * np.abs(x).max()


def test_spmm_of_the_last_rows_one_launch_takes(device):
    # one row to a wavefront: 2^24 - 1 workgroups, which the eighths would round up to
    # 2^24 and beyond a launch; four rows more are refused
    import torch
    from paper_1506_06829_amd import gplhr as G
    n, b = 4 * ((1 << 24) - 1), 33
    rp = torch.arange(n + 5, dtype=torch.int32, device=device)
    ci = rp[:n].flip(0).contiguous()
    v = torch.full((n + 4,), 2.0, dtype=torch.complex64, device=device)
    X = torch.empty((n, b), dtype=torch.complex64, device=device)
    X[:] = rp[:n, None].remainder(8191)
    A = G.DeviceCsr(n, rp[:n + 1], ci, v[:n])
    Y = G.spmm(A, X, val=v[:n])
    for i in (0, 1, 3, n // 2, n - 4, n - 1):
        assert bool((Y[i] == 2.0 * ((n - 1 - i) % 8191)).all()), i
    assert bool((Y[:, b - 1] == 2.0 * ci.remainder(8191)).all())
    del X, Y
    with pytest.raises(G.GplhrError):
        G.spmm(G.DeviceCsr(n + 4, rp, torch.zeros(n + 4, dtype=torch.int32, device=device), v),
               torch.empty((n + 4, b), dtype=torch.complex64, device=device), val=v)


@pytest.mark.parametrize("ld", [1 << 28, (1 << 28) + 1, 1 << 30])
def test_spmm_of_rows_further_apart_than_32_bits(device, ld):
    # a row stride of 2^32 bytes and more (17 GB in all)
    import torch
    from paper_1506_06829_amd import gplhr as G
    n, b = (2, 3) if ld == 1 << 30 else (5, 3)
    rng = np.random.default_rng(6)
    A = sp.csr_matrix(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))
    dA = G.DeviceCsr.from_host(problems.csr_from_scipy(A))
    x = _block(rng, n, b)
    X = torch.empty((n - 1) * ld + b, dtype=torch.complex128, device=device).as_strided((n, b), (ld, 1))
    X.copy_(torch.as_tensor(x))
    Y = G.spmm(dA, X).cpu().numpy()
    assert np.all(np.abs(Y - A @ x) <= 4 * (n + 2) * 2.3e-16 * (abs(A) @ np.abs(x)))


@pytest.mark.parametrize("bx,by", [(1, 1), (5, 10), (10, 10), (16, 16), (30, 48), (48, 48), (64, 64),
                                   (40, 40), (40, 30), (40, 24), (33, 37)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 7, 1000, 100003])
def test_gram_matches_definition(device, bx, by, dtype, n):
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(bx * 100 + by)
    X = _block(rng, n, bx)
    Y = _block(rng, n, by)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    if dtype == "c64":
        X = X.astype(np.complex64).astype(np.complex128)
        Y = Y.astype(np.complex64).astype(np.complex128)
    Xd, Yd = torch.as_tensor(X).to(device, tdt), torch.as_tensor(Y).to(device, tdt)
    Gm = G.gram(Xd, Yd).cpu().numpy()
    ref = X.conj().T @ Y
    scale = np.abs(X).T @ np.abs(Y)
    assert np.max(np.abs(Gm - ref) / scale) < 1e-13     # FP64 accumulation in both dtypes
    assert np.array_equal(Gm, G.gram(Xd, Yd).cpu().numpy())


@pytest.mark.parametrize("w", [1, 8, 10, 16, 24, 32, 40])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gram_of_one_block(device, w, dtype):
    # X^H X with the same block passed on both sides: bitwise the result for
    # a copy on one side, and equal to the definition
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    g = torch.Generator(device="cpu").manual_seed(w)
    for n in ((1000, 100003, (1 << 20) + 37) if w in (10, 32) else (1000, 100003)):
        Xd = torch.randn(n, w + 3, dtype=tdt, generator=g).to(device)[:, 1:w + 1]
        Gs = G.gram(Xd, Xd).cpu().numpy()
        Gc = G.gram(Xd, Xd.clone()).cpu().numpy()
        assert np.array_equal(Gs, Gc), n
        X = Xd.cpu().numpy().astype(np.complex128)
        ref = X.conj().T @ X
        assert np.max(np.abs(Gs - ref) / (np.abs(X).T @ np.abs(X))) < 1e-13


@pytest.mark.parametrize("bx,by", [(64, 64), (48, 48), (32, 32), (64, 16), (40, 16), (48, 10), (40, 40),
                                   (64, 48), (16, 48), (10, 40), (16, 64), (16, 17), (56, 40), (64, 33)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gram_tall_blocks(device, bx, by, dtype):
    # from 2^20 rows the wide tile sets run in their two-waves-per-SIMD build
    # with 512 blocks, Y wider than 32 columns against wide X in the
    # LDS-staged kernel, and X of at most 16 columns against a wider Y as the
    # conjugate transpose of Y^H X; a ragged row count past the threshold
    import torch
    from paper_1506_06829_amd import gplhr as G
    n = (1 << 20) + 37
    g = torch.Generator(device="cpu").manual_seed(bx * 100 + by)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    Xd = torch.randn(n, bx, dtype=tdt, generator=g).to(device)
    Yd = torch.randn(n, by, dtype=tdt, generator=g).to(device)
    Gm = G.gram(Xd, Yd).cpu().numpy()
    X = Xd.cpu().numpy().astype(np.complex128)
    Y = Yd.cpu().numpy().astype(np.complex128)
    ref = X.conj().T @ Y
    scale = np.abs(X).T @ np.abs(Y)
    assert np.max(np.abs(Gm - ref) / scale) < 1e-13
    assert np.array_equal(Gm, G.gram(Xd, Yd).cpu().numpy())


@pytest.mark.parametrize("wy,w", [(0, 9), (0, 48), (0, 64), (1, 7), (8, 8), (9, 15), (20, 44), (16, 48),
                                  (48, 16), (57, 7)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gram_against_own_columns(device, wy, w, dtype):
    # [Y X]^H X with X the last columns of the same block: the shared-operand
    # kernel, at unit and tile edges, with row counts around a K step, a wave's
    # steps and a row block.  Each entry sums n products of FP64 accuracy:
    # n eps of the sum of moduli bounds it.
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    g = torch.Generator(device="cpu").manual_seed(wy * 100 + w)
    for n in (1, 3, 5, 63, 65, 129, 8195, 33001):
        Z = torch.randn(n, wy + w + 2, dtype=tdt, generator=g).to(device)[:, 1:wy + w + 1]
        Gm = G.gram(Z, Z[:, wy:]).cpu().numpy()
        Zh = Z.cpu().numpy().astype(np.complex128)
        ref = Zh.conj().T @ Zh[:, wy:]
        scale = np.abs(Zh).T @ np.abs(Zh[:, wy:])
        assert np.max(np.abs(Gm - ref) / scale) < 4 * (n + 4) * 2.3e-16, n
        assert np.array_equal(Gm[wy:], Gm[wy:].conj().T), n


@pytest.mark.parametrize("bx,by", [(49, 49), (56, 56), (53, 40), (49, 48), (64, 33), (64, 49), (50, 63)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gram_of_odd_unit_counts(device, bx, by, dtype):
    # halves of an odd number of 8-column units overlap in the middle one; the
    # last rows end the allocation.  Bound as above: n products per entry.
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    g = torch.Generator(device="cpu").manual_seed(bx * 100 + by)
    for n in (1, 3, 63, 65, 33001):
        Xd = torch.randn(n, bx, dtype=tdt, generator=g).to(device)
        Yd = torch.randn(n, by, dtype=tdt, generator=g).to(device)
        Gm = G.gram(Xd, Yd).cpu().numpy()
        X, Y = Xd.cpu().numpy().astype(np.complex128), Yd.cpu().numpy().astype(np.complex128)
        scale = np.abs(X).T @ np.abs(Y)
        assert np.max(np.abs(Gm - X.conj().T @ Y) / scale) < 4 * (n + 4) * 2.3e-16, n


@pytest.mark.parametrize("bx,by,own", [(47, 21, False), (18, 41, False), (39, 29, False), (49, 24, False),
                                       (57, 17, False), (45, 45, True), (43, 36, True), (46, 30, True), (62, 22, True)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gram_of_18_to_24_tiles(device, bx, by, own, dtype):
    # up to 21 tiles of two blocks one wave holds all of them, else two share them: row
    # counts around a K step, a wave's steps and a row block.  Bound as above:
    # n products per entry.
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    g = torch.Generator(device="cpu").manual_seed(bx * 100 + by)
    for n in (2049, 2051, 8195, 33001):
        Xd = torch.randn(n, bx, dtype=tdt, generator=g).to(device)
        Yd = Xd[:, bx - by:] if own else torch.randn(n, by, dtype=tdt, generator=g).to(device)
        Gm = G.gram(Xd, Yd).cpu().numpy()
        X, Y = Xd.cpu().numpy().astype(np.complex128), Yd.cpu().numpy().astype(np.complex128)
        scale = np.abs(X).T @ np.abs(Y)
        assert np.max(np.abs(Gm - X.conj().T @ Y) / scale) < 4 * (n + 4) * 2.3e-16, n
        assert np.array_equal(Gm, G.gram(Xd, Yd).cpu().numpy()), n


@pytest.mark.parametrize("bx,by,own", [(17, 9, False), (9, 17, False), (64, 64, False), (40, 16, True), (20, 20, True)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_gram_of_few_rows(device, bx, by, own, dtype):
    # one workgroup per tile over all rows: row counts around a wavefront's steps
    # and around the sizes at which the kernels with partials take over.  Bound
    # as above: n products per entry.
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    g = torch.Generator(device="cpu").manual_seed(bx * 100 + by)
    for n in (2, 61, 64, 449, 452, 513, 963, 1024, 1025, 2047, 2048, 2049):
        Xd = torch.randn(n, bx, dtype=tdt, generator=g).to(device)
        Yd = Xd[:, bx - by:] if own else torch.randn(n, by, dtype=tdt, generator=g).to(device)
        Gm = G.gram(Xd, Yd).cpu().numpy()
        X, Y = Xd.cpu().numpy().astype(np.complex128), Yd.cpu().numpy().astype(np.complex128)
        scale = np.abs(X).T @ np.abs(Y)
        assert np.max(np.abs(Gm - X.conj().T @ Y) / scale) < 4 * (n + 4) * 2.3e-16, n
        assert np.array_equal(Gm, G.gram(Xd, Yd.clone() if own and bx == by else Yd).cpu().numpy()), n


def test_gram_of_rows_far_apart(device):
    # a leading dimension whose rows lie further apart than the kernels' 32-bit
    # offsets reach
    import torch
    from paper_1506_06829_amd import gplhr as G
    ld, n = 90_000_000, 3
    X = torch.zeros((n - 1) * ld + 8, dtype=torch.complex128, device=device).as_strided((n, 5), (ld, 1))
    x = torch.randn(n, 5, dtype=torch.complex128, generator=torch.Generator().manual_seed(3))
    X.copy_(x)
    Gm = G.gram(X, X[:, 2:4]).cpu().numpy()
    ref = x.numpy().conj().T @ x.numpy()[:, 2:4]
    assert np.max(np.abs(Gm - ref)) < 1e-14 * np.max(np.abs(ref)) * n


@pytest.mark.parametrize("wx,wy", [(1, 1), (7, 5), (10, 10), (16, 16), (40, 20), (30, 10), (10, 30),
                                   (64, 32), (64, 16), (48, 48), (16, 48), (33, 40), (128, 8)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("beta", [0.0, 1.0, 0.5 - 0.25j])
def test_block_update_matches_definition(device, wx, wy, dtype, beta):
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(wx * 64 + wy)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    for n in (1, 17, 1000, 100003):
        X = _block(rng, n, wx, ld=wx + 3)
        Y0 = _block(rng, n, wy, ld=wy + 2)
        M = rng.standard_normal((wx, wy)) + 1j * rng.standard_normal((wx, wy))
        if dtype == "c64":
            X = X.astype(np.complex64).astype(np.complex128)
            Y0 = Y0.astype(np.complex64).astype(np.complex128)
        Xd = torch.as_tensor(X).to(device, tdt)[:, :wx]          # strided blocks
        Yfull = torch.as_tensor(Y0).to(device, tdt)
        Md = torch.as_tensor(M).to(device)
        out = G.block_update(Xd, Md, Yfull[:, :wy], beta=beta).cpu().numpy()
        ref = beta * Y0[:, :wy] + X[:, :wx] @ M
        scale = abs(beta) * np.abs(Y0[:, :wy]) + np.abs(X[:, :wx]) @ np.abs(M)
        tol = 1e-14 if dtype == "c128" else 3e-6
        assert np.max(np.abs(out - ref) / scale) < tol, (n, wx, wy)
        # the columns past wy are left alone
        rest = Yfull[:, wy:].cpu().numpy()
        assert np.array_equal(rest, Y0[:, wy:].astype(rest.dtype))


@pytest.mark.parametrize("wx,wy", [(16, 16), (32, 16), (48, 16), (64, 16), (16, 48), (64, 32), (64, 48),
                                   (8, 8), (40, 24), (6, 10), (2, 2)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("beta", [0.0, 1.0, 0.5 - 0.25j])
def test_block_update_even_strides(device, wx, wy, dtype, beta):
    # even widths and leading dimensions: the shapes the pipelined kernel
    # takes for complex64 too (16-byte pairs and output chunks), with the
    # output inside a wider block and rows in ragged counts
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(wx * 64 + wy + 7)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    for n in (1, 17, 1000, 100003):
        X = _block(rng, n, wx, ld=wx + 4)
        Y0 = _block(rng, n, wy, ld=wy + 6)
        M = rng.standard_normal((wx, wy)) + 1j * rng.standard_normal((wx, wy))
        if dtype == "c64":
            X = X.astype(np.complex64).astype(np.complex128)
            Y0 = Y0.astype(np.complex64).astype(np.complex128)
        Xd = torch.as_tensor(X).to(device, tdt)[:, 2:wx + 2]
        Yfull = torch.as_tensor(Y0).to(device, tdt)
        Md = torch.as_tensor(M).to(device)
        out = G.block_update(Xd, Md, Yfull[:, 4:wy + 4], beta=beta).cpu().numpy()
        ref = beta * Y0[:, 4:wy + 4] + X[:, 2:wx + 2] @ M
        scale = abs(beta) * np.abs(Y0[:, 4:wy + 4]) + np.abs(X[:, 2:wx + 2]) @ np.abs(M)
        tol = 1e-14 if dtype == "c128" else 3e-6
        assert np.max(np.abs(out - ref) / scale) < tol, (n, wx, wy)
        rest = Yfull.cpu().numpy()
        assert np.array_equal(rest[:, :4], Y0[:, :4].astype(rest.dtype))
        assert np.array_equal(rest[:, wy + 4:], Y0[:, wy + 4:].astype(rest.dtype))


@pytest.mark.parametrize("wx,wy,off", [(1, 1, 0), (9, 9, 0), (8, 16, 1), (16, 24, 0), (24, 17, 1), (41, 33, 0),
                                       (42, 42, 0), (57, 40, 1), (64, 48, 0)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("beta", [0.0, -0.5 + 1.0j])
def test_block_update_row_groups(device, wx, wy, off, dtype, beta):
    # row counts around a row group and a workgroup's groups, ragged slabs and
    # tiles, blocks inside NaN-filled storage at even and odd column offsets:
    # nothing outside the block is read into a result or written.  wx products
    # and beta Y per entry: (wx + 4) eps of the sum of moduli bounds each part.
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt, eps = (torch.complex128, 2.3e-16) if dtype == "c128" else (torch.complex64, 1.2e-7)
    g = torch.Generator(device="cpu").manual_seed(wx * 100 + wy)
    nan = complex(float("nan"), float("nan"))
    for n in (1, 15, 17, 33, 64, 129, 4097, 33003):
        Xs = torch.full((n, wx + 4), nan, dtype=tdt)
        Ys = torch.full((n, wy + 4), nan, dtype=tdt)
        Xs[:, off:off + wx] = torch.randn(n, wx, dtype=tdt, generator=g)
        Ys[:, off:off + wy] = torch.randn(n, wy, dtype=tdt, generator=g)
        if n > 20:
            Xs[7, off] = complex(float("inf"), 0.0)      # one bad row stays one
        M = torch.randn(wx, wy, dtype=torch.complex128, generator=g)
        Xd, Yd = Xs.to(device), Ys.to(device)
        G.block_update(Xd[:, off:off + wx], M.to(device), Yd[:, off:off + wy], beta=beta)
        out = Yd.cpu().numpy()
        x = Xs[:, off:off + wx].numpy().astype(np.complex128)
        y = Ys[:, off:off + wy].numpy().astype(np.complex128)
        rows = np.ones(n, bool)
        if n > 20:
            rows[7] = False
            assert not np.isfinite(out[7, off:off + wy]).any()
        with np.errstate(invalid="ignore"):
            ref = beta * y + x @ M.numpy()
            scale = abs(beta) * np.abs(y) + np.abs(x) @ np.abs(M.numpy())
        err = np.abs(out[:, off:off + wy] - ref)[rows] / scale[rows]
        assert err.max() < 2 * (wx + 4) * eps, n
        assert np.isnan(out[:, :off]).all() and np.isnan(out[:, off + wy:]).all()


@pytest.mark.parametrize("wx,wy,pad", [(3, 47, 0), (7, 30, 6), (6, 32, 0), (20, 15, 1), (33, 31, 3), (57, 13, 6), (16, 30, 2),
                                       (64, 33, 0), (40, 10, 30), (64, 32, 0)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_block_update_beyond_the_caches(device, wx, wy, pad, dtype):
    # outputs over 256 MiB: rows that leave in runs or in pieces, with and without gaps,
    # on and off cache lines; what lies between the rows stays.  wx products per entry:
    # (wx + 4) eps of the sum of moduli, on the GPU's rows sampled from all parts.
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt, eps, size = (torch.complex128, 2.3e-16, 16) if dtype == "c128" else (torch.complex64, 1.2e-7, 8)
    g = torch.Generator(device=device).manual_seed(wx * 100 + wy)
    n = (256 << 20) // (wy * size) + 1003
    X = torch.randn(n, wx + pad, dtype=tdt, device=device, generator=g)
    Y = torch.full((n, wy + pad), 7.0, dtype=tdt, device=device)
    M = torch.randn(wx, wy, dtype=torch.complex128, device=device, generator=g)
    out = Y[:, pad // 2:pad // 2 + wy]
    G.block_update(X[:, :wx], M, out)
    rows = torch.cat([torch.arange(0, 2000), torch.arange(n - 2000, n), torch.randint(0, n, (4000,))]).to(device)
    x, o = X[rows, :wx].to(torch.complex128).cpu().numpy(), out[rows].to(torch.complex128).cpu().numpy()
    m = M.cpu().numpy()
    assert np.max(np.abs(o - x @ m) / (np.abs(x) @ np.abs(m))) < 2 * (wx + 4) * eps
    assert bool((Y[:, :pad // 2] == 7.0).all()) and bool((Y[:, pad // 2 + wy:] == 7.0).all())
    if pad == 0:    # the rows between the sampled ones: against the same rows as a small block
        k = n // 3
        part = torch.empty(20000, wy, dtype=tdt, device=device)
        G.block_update(X[k:k + 20000].clone(), M, part)
        assert bool(((part - out[k:k + 20000]).abs() <= 2 * (wx + 4) * eps * 64 * wx).all())


@pytest.mark.parametrize("wy,w,dtype", [(15, 16, "c128"), (14, 18, "c64"), (9, 24, "c128")])
def test_proj_orth_beyond_the_caches(device, wy, w, dtype):
    # updates by a triangular factor whose outputs leave in runs, in place
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt, eps, size = (torch.complex128, 2.3e-16, 16) if dtype == "c128" else (torch.complex64, 1.2e-7, 8)
    g = torch.Generator(device=device).manual_seed(wy)
    n = (256 << 20) // (w * size) + 777
    Z = torch.randn(n, wy + w, dtype=tdt, device=device, generator=g)
    G.proj_orth(Z[:, :wy], 0, wy)
    Y = Z[:, :wy].clone()
    G.proj_orth(Z, wy, w)
    H = G.gram(Z, Z).cpu().numpy()
    assert torch.equal(Z[:, :wy], Y)
    assert np.max(np.abs(H - np.eye(wy + w))) < 100 * eps


@pytest.mark.parametrize("w", [10, 16, 48])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_block_update_in_place(device, w, dtype):
    # Y = X itself (the Cholesky-QR normalisation W <- W R^-1 is done this way)
    import torch
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(w)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    n = 100003
    X = _block(rng, n, w)
    if dtype == "c64":
        X = X.astype(np.complex64).astype(np.complex128)
    M = np.triu(rng.standard_normal((w, w)) + 1j * rng.standard_normal((w, w))) + 3 * np.eye(w)
    Xd = torch.as_tensor(X).to(device, tdt)
    G.block_update(Xd, torch.as_tensor(M).to(device), Xd)
    ref = X @ M
    scale = np.abs(X) @ np.abs(M)
    tol = 1e-14 if dtype == "c128" else 3e-6
    assert np.max(np.abs(Xd.cpu().numpy() - ref) / scale) < tol


@pytest.mark.parametrize("wy,w", [(0, 16), (16, 16), (16, 48), (0, 48), (48, 16), (32, 32),
                                  (10, 20), (3, 5), (24, 40), (8, 48)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_proj_orth_matches_qr(device, wy, w, dtype):
    # Z(:, wy:wy+w) <- orth((I - Y Y^H) X) in two passes: the Q of the QR
    # factorisation of the projected block with a positive real diagonal (the
    # oracle's orth); Y = Z(:, :wy) and the columns after the block are left
    # as they were.  The 48-column blocks take the update path that skips the
    # zero products of the triangular R^{-1}.
    import torch
    from oracle.gplhr_oracle import orth
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(100 * wy + w)
    tdt = torch.complex128 if dtype == "c128" else torch.complex64
    for n in (257, 100003):
        ld = wy + w + 2
        Z = _block(rng, n, ld)
        if wy:
            Z[:, :wy] = orth(Z[:, :wy])
            # a component along Y for the projection to remove
            Z[:, wy:wy + w] += Z[:, :wy] @ (rng.standard_normal((wy, w)) + 1j * rng.standard_normal((wy, w)))
        if dtype == "c64":
            Z = Z.astype(np.complex64).astype(np.complex128)
        Y, X = Z[:, :wy], Z[:, wy:wy + w]
        ref = orth(X - Y @ (Y.conj().T @ X))
        Zd = torch.as_tensor(Z).to(device, tdt)
        G.proj_orth(Zd, wy, w, passes=2)
        out = Zd.cpu().numpy().astype(np.complex128)
        tol = 1e-12 if dtype == "c128" else 2e-5
        err = np.linalg.norm(out[:, wy:wy + w] - ref) / np.sqrt(w)
        assert err < tol, (n, wy, w, err)
        Q = out[:, wy:wy + w]
        assert np.max(np.abs(Q.conj().T @ Q - np.eye(w))) < (1e-13 if dtype == "c128" else 1e-5)
        if wy:
            assert np.max(np.abs(Y.conj().T @ Q)) < (1e-13 if dtype == "c128" else 1e-5)
        assert np.array_equal(out[:, :wy], Z[:, :wy])
        assert np.array_equal(out[:, wy + w:], Z[:, wy + w:])


@pytest.mark.parametrize("wy,w", [(0, 1), (7, 1), (0, 15), (1, 17), (31, 31), (31, 33), (17, 47), (48, 15)])
def test_proj_orth_factor_tiles(device, wy, w):
    # widths around the factor's 16-column tiles and its largest G_Y, with a
    # block of condition number 1e3: the first pass's orthogonality loss stays
    # far below one, so the second leaves n eps, and Q differs from the oracle's
    # by no more than cond * n eps
    import torch
    from oracle.gplhr_oracle import orth
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(100 * wy + w)
    n = 300
    Z = _block(rng, n, wy + w + 1)
    if wy:
        Z[:, :wy] = orth(Z[:, :wy])
    U = np.linalg.qr(rng.standard_normal((w, w)))[0]
    Z[:, wy:wy + w] = Z[:, wy:wy + w] @ (U * np.logspace(0, -3, w)) @ U.T
    Y, X = Z[:, :wy], Z[:, wy:wy + w]
    ref = orth(X - Y @ (Y.conj().T @ X))
    Zd = torch.as_tensor(Z).to(device)
    G.proj_orth(Zd, wy, w, passes=2)
    out = Zd.cpu().numpy()
    Q = out[:, wy:wy + w]
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(w))) < n * 2.3e-16
    assert np.linalg.norm(Q - ref) / np.sqrt(w) < 1e3 * n * 2.3e-16
    assert np.array_equal(out[:, :wy], Z[:, :wy]) and np.array_equal(out[:, wy + w:], Z[:, wy + w:])


@pytest.mark.parametrize("wy", [0, 16])
def test_proj_orth_reports_rank_deficiency(device, wy):
    # a column that repeats another leaves a vanishing Cholesky pivot:
    # BREAKDOWN, not a silent result
    import torch
    from oracle.gplhr_oracle import orth
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(5 + wy)
    n, w = 4099, 16
    Z = _block(rng, n, wy + w)
    if wy:
        Z[:, :wy] = orth(Z[:, :wy])
    Z[:, wy + 7] = Z[:, wy + 2]
    Zd = torch.as_tensor(Z).to(device)
    with pytest.raises(Exception, match="rank deficient"):
        G.proj_orth(Zd, wy, w, passes=2)


def test_proj_orth_column_inside_span_y(device):
    # a column inside span(Y): the first pass only projects (the cancellation
    # guard), the second normalises what is left, so the column comes back as
    # a unit vector orthogonal to Y and to the other columns
    import torch
    from oracle.gplhr_oracle import orth
    from paper_1506_06829_amd import gplhr as G
    rng = np.random.default_rng(11)
    n, wy, w = 4099, 16, 16
    Z = _block(rng, n, wy + w)
    Z[:, :wy] = orth(Z[:, :wy])
    Z[:, wy + 3] = Z[:, :wy] @ rng.standard_normal(wy)
    Zd = torch.as_tensor(Z).to(device)
    G.proj_orth(Zd, wy, w, passes=2)
    Q = Zd.cpu().numpy()[:, wy:]
    assert np.max(np.abs(Q.conj().T @ Q - np.eye(w))) < 1e-13
    assert np.max(np.abs(Z[:, :wy].conj().T @ Q)) < 1e-13
    # the other columns are those of the QR factorisation with that column
    # taken out of the block
    keep = [c for c in range(w) if c != 3]
    X = Z[:, wy:][:, keep]
    ref = orth(X - Z[:, :wy] @ (Z[:, :wy].conj().T @ X))
    assert np.linalg.norm(Q[:, [0, 1, 2]] - ref[:, :3]) < 1e-12


def test_block_update_rejects_oversized_coefficients(device):
    import torch
    from paper_1506_06829_amd import gplhr as G
    X = torch.zeros((64, 128), dtype=torch.complex128, device=device)
    M = torch.zeros((128, 48), dtype=torch.complex128, device=device)
    with pytest.raises(Exception, match="LDS"):
        G.block_update(X, M)


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n,w,ldx,ldy", [(1, 2, 2, 2), (1000003, 16, 16, 16), (4099, 6, 10, 8)])
def test_block_copy(device, dtype, n, w, ldx, ldy):
    # the streaming block copy: Y(:, 0:w) = X(:, 0:w), columns beyond w of Y
    # untouched, contiguous and strided rows
    import torch
    from paper_1506_06829_amd import gplhr as G
    tdt = getattr(torch, dtype)
    X = torch.randn(n, ldx, dtype=tdt, device="cuda")
    Y = torch.full((n, ldy), 7.0, dtype=tdt, device="cuda")
    G.block_copy(X[:, :w], Y[:, :w])
    torch.cuda.synchronize()
    assert torch.equal(Y[:, :w], X[:, :w])
    assert bool((Y[:, w:] == 7.0).all())
