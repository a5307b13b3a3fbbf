"""Resident solves (matrix kept in registers, one cooperative launch) against
the CPU oracle, at the sizes where their launch shape changes.

Bounds: the systems are diagonally dominant (their Jacobi-scaled rows sum to at
most 1/2 off the diagonal), so three iterations amplify the rounding of a dot
over n terms (below 1e-13 relative for n up to 4e5) and of a row by less than
ten: complex128 iterates within 1e-11 of the oracle's.  complex64 iterates differ
by the rounding of their vectors, 2^-24 per operation over some thirty
operations: 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def hk():
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_2112_11880_amd as hk
    hk.load()
    return hk


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def crandn(rng, n):
    return rng.standard_normal(n) + 1j * rng.standard_normal(n)


def dominant(n, row, seed):
    """Rows of 1 to `row` entries (the longest included), columns near and far from the diagonal."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, row + 1, n)
    lens[: max(1, n // 2)] = row
    k = max(row - 1, 1)
    off = np.where(rng.random((n, k)) < 0.7, rng.integers(-40, 41, (n, k)), rng.integers(-n, n + 1, (n, k)))
    off[0] = np.arange(1, k + 1)  # the one row that surely has no column twice
    col = np.clip(np.arange(n)[:, None] + off, 0, n - 1)
    col[np.arange(k)[None, :] >= lens[:, None] - 1] = -1
    col = np.concatenate([col, np.arange(n)[:, None]], axis=1)
    col.sort(axis=1)
    keep = col >= 0
    keep[:, 1:] &= col[:, 1:] != col[:, :-1]
    cnt = keep.sum(1)
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(cnt)
    cols = col[keep].astype(np.int32)
    val = crandn(rng, cols.shape[0]) / (4.0 * row)
    val[cols == np.repeat(np.arange(n), cnt)] = 1.0 + 0.25 * crandn(rng, n)
    return rowptr, cols, val, crandn(rng, n)


# (rows, longest row, shape's rows per thread and waves, or None: the system does not fit)
SHAPES = [
    (1, 1, (1, 4)), (63, 8, (1, 4)), (64, 9, (1, 4)), (65, 15, (1, 4)), (257, 16, (1, 4)), (300, 27, (1, 4)),
    (300, 28, None), (16384, 15, (1, 4)), (16385, 15, (1, 8)), (16385, 27, (1, 8)),
    (131072, 15, (1, 8)), (131073, 15, (2, 8)), (131073, 8, (2, 8)), (131073, 27, None),
    (262144, 15, (2, 8)), (262145, 15, None),
]


@pytest.mark.parametrize("n,row,shape", SHAPES)
@pytest.mark.parametrize("method", ["bicgstab", "tfqmr"])
def test_resident_iterates(hk, oracle, n, row, shape, method):
    print("[case]", method, n, row, flush=True)
    rowptr, col, val, b = dominant(n, row, n + row)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    ref = oracle.bicgstab if method == "bicgstab" else oracle.tfqmr
    for k in (1, 3):
        x, info, hist = hk.krylov_solve(A, dev(b), tol=0.0, max_iter=k, method=method, history=True)
        xo, oi, ho = ref(rowptr, col, val, b, tol=0.0, maxit=k, history=True)
        if n > 1:
            assert info["status"] == oi["status"] == hk.HK_NOT_CONVERGED and info["iters"] == k, (info, oi)
            assert np.allclose(hist.cpu().numpy(), ho, rtol=1e-9, atol=0)
        if shape is not None:
            assert info["shape"][0] == 1 and tuple(info["shape"][1:3]) == shape, info["shape"]
        else:
            assert info["shape"][0] != 1, info["shape"]
        assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-11 * np.linalg.norm(xo)


@pytest.mark.parametrize("n,row,shape", [(1, 1, (1, 4)), (65, 8, (1, 4)), (300, 27, (1, 4)), (300, 28, None), (6000, 15, (1, 4)),
                                         (16385, 15, (1, 8)), (16385, 8, (1, 8)), (20000, 27, (1, 8)), (131073, 8, (2, 8)),
                                         (131073, 15, (2, 8))])
@pytest.mark.parametrize("ell,cycles", [(1, 3), (2, 2), (4, 1)])
def test_resident_bicgstab_l_iterates(hk, oracle, n, row, shape, ell, cycles):
    """The minimal-residual coefficients carry the rounding times the condition
    of the Gram matrix of r_1 .. r_l, whose vectors lie within 1/2 of each other's
    directions (below 1e5 for l <= 4); they scale a correction of the size of the
    residual, 1e-2 of the start's by then.  l = 8 is not compared here: eight steps
    solve these systems, and the oracle's own iterate then changes by 1e6 to 1e10
    times a change of b (test_resident_bicgstab_8_solves)."""
    print("[case] bicgstab_l", ell, n, row, flush=True)
    rowptr, col, val, b = dominant(n, row, n + row)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    x, info = hk.krylov_solve(A, dev(b), tol=1e-12 if n == 1 else 0.0, max_iter=cycles, method="bicgstab_l", ell=ell)
    xo, oi = oracle.bicgstab_l(rowptr, col, val, b, ell=ell, tol=1e-12 if n == 1 else 0.0, maxit=cycles)
    assert info["status"] == oi["status"] and info["iters"] == oi["iters"], (info, oi)
    assert (tuple(info["shape"][:3]) == (1, *shape)) if shape else info["shape"][0] != 1, info["shape"]
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)


@pytest.mark.parametrize("cells,rpt", [((9, 8, 7), 1), ((30, 29, 31), 1), ((60, 45, 50), 2)])
def test_resident_bicgstab_8_solves(hk, oracle, cells, rpt):
    """Meshes of 720, 28,800+ and 143,106 rows, many cycles: the oracle's residual
    of the solution is the one reported and meets the tolerance, and the monitored
    residual has not left it by more than the rounding that l = 8 gathers."""
    from synth import helmholtz as H
    print("[case] bicgstab(8)", cells, flush=True)
    m = H.make_mesh(*cells, 1.0 / max(cells), jitter=0.2, rng=np.random.default_rng(3))
    p = H.build_problem(m)
    val = H.helmholtz_values(p, complex(9.0, 0.09))
    b = H.complex_rhs(np.random.default_rng(0), p.n, p.dirichlet)
    x, info = hk.krylov_solve(hk.CSR(dev(p.rowptr), dev(p.col), dev(val)), dev(b), tol=1e-8, method="bicgstab_l", ell=8)
    assert info["status"] == hk.HK_OK and info["iters"] > 1 and info["shape"][:2] == [1, rpt], info
    r = oracle.residual(p.rowptr, p.col, val, b, x.cpu().numpy())
    rel = np.linalg.norm(r) / np.linalg.norm(b)
    assert rel <= 1.05e-8 and abs(rel - info["relres_true"]) <= 1e-10 and info["relres_rec"] <= 1e-8


@pytest.mark.parametrize("n,row,rpt", [(1000, 8, 1), (16385, 15, 1), (131073, 15, 2), (262145, 15, 3), (393217, 15, 4),
                                       (131072, 27, 1), (131073, 27, 2), (262145, 8, 3), (393217, 8, 4)])
def test_resident_complex64_iterates(hk, oracle, n, row, rpt):
    print("[case] complex64", n, row, flush=True)
    rowptr, col, val, b = dominant(n, row, n + row)
    v32, b32 = val.astype(np.complex64), b.astype(np.complex64)
    x, info = hk.krylov_solve(hk.CSR(dev(rowptr), dev(col), dev(v32)), dev(b32), tol=0.0, max_iter=3)
    xo, oi = oracle.bicgstab_c64(rowptr, col, v32, b32, tol=0.0, maxit=3)
    assert info["iters"] == oi["iters"] == 3 and info["shape"][:2] == [1, rpt], info
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-5 * np.linalg.norm(xo)


@pytest.mark.parametrize("method", ["bicgstab", "tfqmr"])
def test_resident_options_and_fallback(hk, oracle, monkeypatch, method):
    """x0, no preconditioner, a solve to its tolerance, and the same solve by
    the separate kernels: a handle with a fixed plan uses them, and so does a
    resident launch whose barrier waits are not allowed to take any time."""
    rowptr, col, val, b = dominant(5000, 15, 9)
    rng = np.random.default_rng(1)
    x0 = crandn(rng, 5000)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    B = hk.CSR(dev(rowptr), dev(col), dev(val))
    B.set_plan(64, 32, 0)
    ref = oracle.bicgstab if method == "bicgstab" else oracle.tfqmr
    for kw, okw in (({"x": dev(x0)}, {"x0": x0}), ({"precond": False}, {"precond": False})):
        print("[case]", method, sorted(kw), flush=True)
        x, info = hk.krylov_solve(A, dev(b), tol=0.0, max_iter=2, method=method, **kw)
        xo, _ = ref(rowptr, col, val, b, tol=0.0, maxit=2, **okw)
        assert info["shape"][0] == 1
        assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-11 * np.linalg.norm(xo)
    x, info = hk.krylov_solve(A, dev(b), tol=1e-12, method=method)
    y, other = hk.krylov_solve(B, dev(b), tol=1e-12, method=method)
    assert info["status"] == other["status"] == hk.HK_OK and info["shape"][0] == 1 and other["shape"][0] == 64
    r = oracle.residual(rowptr, col, val, b, x.cpu().numpy())
    assert np.linalg.norm(r) <= 1.05e-12 * np.linalg.norm(b) and info["relres_true"] <= 1.05e-12
    assert torch.equal(x, hk.krylov_solve(A, dev(b), tol=1e-12, method=method)[0])
    print("[case]", method, "barrier limit of one tick", flush=True)
    monkeypatch.setenv("HK_BARRIER_SPIN_TICKS", "1")
    C = hk.CSR(dev(rowptr), dev(col), dev(val))
    z, late = hk.krylov_solve(C, dev(b), x=dev(x0), tol=1e-12, method=method)
    assert late["status"] == hk.HK_OK and late["shape"][0] == 64, late
    assert (z - x).abs().max() <= 1e-10 * x.abs().max()


def block_diagonal(sizes, row, seed):
    parts = [dominant(n, min(row, n), seed + k) for k, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)])
    nnz = np.cumsum([0] + [p[1].shape[0] for p in parts])
    rowptr = np.concatenate([[0]] + [p[0][1:] + z for p, z in zip(parts, nnz)]).astype(np.int32)
    col = np.concatenate([p[1] + o for p, o in zip(parts, off)]).astype(np.int32)
    return parts, off, rowptr, col, np.concatenate([p[2] for p in parts]), np.concatenate([p[3] for p in parts])


@pytest.mark.parametrize("sizes,row", [
    ([1], 1), ([1, 2, 63, 64, 65, 130], 8), ([700, 5, 20000, 513, 1], 15), ([40000, 70000, 3000] + [65] * 61, 15),
    ([131073, 900, 131072, 17], 15), ([500, 9000, 27], 27), ([300, 40], 28),
])
def test_resident_batch(hk, oracle, sizes, row):
    """Systems of 1 row to more than one workgroup takes, several lists deep; a zero
    right-hand side and a NaN each end their system only."""
    print("[case] batch", sizes[:6], row, flush=True)
    parts, off, rowptr, col, val, b = block_diagonal(sizes, row, 17)
    b = b.copy()
    zero = nan = -1
    if len(sizes) > 3:
        zero, nan = 1, 3
        b[off[zero]:off[zero + 1]] = 0
        b[off[nan]] = np.nan
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    for tol, k in ((0.0, 2), (1e-12, 400)):
        x, infos = hk.blockdiag_solve(A, off, dev(b), tol=tol, max_iter=k)
        x = x.cpu().numpy()
        for s, (rp, c, v, _) in enumerate(parts):
            bs, xs, info = b[off[s]:off[s + 1]], x[off[s]:off[s + 1]], infos[s]
            if s == zero:
                assert info["status"] == hk.HK_OK and info["iters"] == 0 and np.all(xs == 0), info
            elif s == nan:
                assert info["status"] == hk.HK_NONFINITE, info
            elif tol:
                assert info["status"] == hk.HK_OK and info["relres_true"] <= 1.05e-12, (s, info)
                r = oracle.residual(rp, c, v, bs, xs)
                assert np.linalg.norm(r) <= 1.05e-12 * np.linalg.norm(bs)
            elif sizes[s] > 4:
                xo, oi = oracle.bicgstab(rp, c, v, bs, tol=0.0, maxit=k)
                assert info["status"] == oi["status"] == hk.HK_NOT_CONVERGED and info["iters"] == k, (s, info, oi)
                assert np.linalg.norm(xs - xo) <= 1e-11 * np.linalg.norm(xo), s
                assert abs(info["relres_true"] - oi["relres_true"]) <= 1e-11, (s, info, oi)


@pytest.mark.parametrize("n,row,nsys", [
    (512, 15, 3), (513, 15, 3), (1000, 8, 64), (9000, 15, 33), (20011, 15, 5), (70001, 15, 7), (131073, 15, 3),
    (140000, 8, 2), (40000, 27, 5), (131073, 27, 2), (3000, 28, 3),
    # several systems at a time in a group: 2 to 8, fewer and more than the queue holds
    (60001, 15, 4), (40001, 15, 64), (131072, 15, 2), (100003, 15, 19), (33000, 8, 13)])
def test_resident_sweep(hk, oracle, n, row, nsys):
    """Sweeps on both sides of the limits: one system per group of workgroups, more systems than groups,
    one and two rows per thread, and systems that do not fit.  Off the diagonal the scaled rows sum to less
    than 1/2 as above."""
    rowptr, col, val, _ = dominant(n, row, n + row)
    rng = np.random.default_rng(n)
    diag = col == np.repeat(np.arange(n), np.diff(rowptr))
    K, M = np.where(diag, 1.0, val.real), np.where(diag, 0.2, val.imag)
    kap = [complex(0.1 + 0.4 * j / nsys, 0.01 * (j + 1)) for j in range(nsys)]
    B = np.zeros((n, 64), dtype=np.complex128)
    for j in range(nsys):
        B[:, j] = crandn(rng, n)
    B[:, nsys - 1] = 0
    args = (dev(rowptr), dev(col), dev(K), dev(M), kap, dev(B))
    for its in (3, 0):
        print("resident sweep", n, row, nsys, its, flush=True)
        X, infos = hk.sweep_solve(*args, tol=1e-14, max_iter=its)
        Xh = X.cpu().numpy()
        for j in range(nsys):
            xo, oi = oracle.bicgstab(rowptr, col, K - kap[j] * M, B[:, j], tol=1e-14, maxit=its)
            assert infos[j]["iters"] == oi["iters"] and infos[j]["status"] == oi["status"], (its, j, infos[j], oi)
            assert np.linalg.norm(Xh[:, j] - xo) <= 1e-11 * np.linalg.norm(xo), (its, j)
            if j < nsys - 1:
                r = oracle.residual(rowptr, col, K - kap[j] * M, B[:, j], Xh[:, j])
                assert abs(np.linalg.norm(r) / np.linalg.norm(B[:, j]) - infos[j]["relres_true"]) <= 1e-12
        assert np.all(Xh[:, nsys:] == 0)
    X, infos = hk.sweep_solve(*args, tol=1e-10)
    X2, _ = hk.sweep_solve(*args, tol=1e-10)
    assert all(i["status"] == 0 and i["relres_true"] <= 1e-9 for i in infos)
    assert torch.equal(torch.view_as_real(X), torch.view_as_real(X2))


def banded(n, dist, seed):
    """Rows with entries at the given distances (clipped at the ends), a few of them left out."""
    rng = np.random.default_rng(seed)
    d = np.array(sorted(set(dist) | {0}))
    col = np.arange(n)[:, None] + d[None, :]
    keep = (col >= 0) & (col < n) & ((rng.random(col.shape) < 0.99) | (d == 0)[None, :])
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(keep.sum(1))
    cols = col[keep].astype(np.int32)
    val = crandn(rng, cols.shape[0]) / (4.0 * len(d))
    val[cols == np.repeat(np.arange(n), keep.sum(1))] = 1.0 + 0.125 * rng.standard_normal(n)
    return rowptr, cols, val, crandn(rng, n)


@pytest.mark.parametrize("n,ndist", [(300007, 15), (262208, 15), (290000, 11), (150001, 27), (40000, 28), (64 * 500 + 1, 33)])
@pytest.mark.parametrize("method", ["bicgstab", "tfqmr", "bicgstab_l", "c64"])
def test_sliced_products(hk, oracle, n, ndist, method):
    """Systems that do not fit the registers and have few distances col - row per 64 rows: the first
    iterates with the sliced products, in a last slice of 1 to 64 rows, whole fives of distances and not."""
    rng = np.random.default_rng(ndist)
    rowptr, col, val, b = banded(n, [0, 1, -1, 70, -70] + list(rng.choice(np.r_[-3000:-100, 100:3000], ndist - 5, replace=False)), n)
    print("[case] slices", n, ndist, method, flush=True)
    its = 2 if method == "bicgstab_l" else 3
    if method == "c64":
        v32, b32 = val.astype(np.complex64), b.astype(np.complex64)
        x, info = hk.krylov_solve(hk.CSR(dev(rowptr), dev(col), dev(v32)), dev(b32), tol=0.0, max_iter=its)
        xo, oi = oracle.bicgstab_c64(rowptr, col, v32, b32, tol=0.0, maxit=its)
        assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-5 * np.linalg.norm(xo)
        assert info["shape"][0] == (2 if ndist > 27 else 1)
        return
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    kw = {"ell": 2} if method == "bicgstab_l" else {}
    xo, oi = getattr(oracle, method)(rowptr, col, val, b, tol=0.0, maxit=its, **kw)
    x, info = hk.krylov_solve(A, dev(b), tol=0.0, max_iter=its, method=method, **kw)
    assert info["shape"] == [2, 64, 4, 0] and info["iters"] == oi["iters"], info
    assert np.linalg.norm(x.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)
    A.set_plan(64, 32)
    y, info = hk.krylov_solve(A, dev(b), tol=0.0, max_iter=its, method=method, **kw)
    assert info["shape"][0] == 64 and np.linalg.norm(y.cpu().numpy() - xo) <= 1e-10 * np.linalg.norm(xo)


def test_resident_batch_and_sweep_are_taken(hk):
    """Without a shape given, the batch and the sweep take the resident launches: their sums run in
    another order than those of the launch in the shape reported, so some bits differ."""
    parts, off, rowptr, col, val, b = block_diagonal([3000, 900, 20000], 15, 5)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    x, infos = hk.blockdiag_solve(A, off, dev(b), tol=1e-12)
    y, _ = hk.blockdiag_solve(A, off, dev(b), tol=1e-12, shape=infos[0]["shape"])
    for k in range(3):
        lo, hi = off[k], off[k + 1]
        assert not torch.equal(x[lo:hi], y[lo:hi]) and torch.allclose(x[lo:hi], y[lo:hi], rtol=1e-9, atol=1e-11)
    rowptr, col, val, _ = dominant(5000, 15, 9)
    diag = col == np.repeat(np.arange(5000), np.diff(rowptr))
    K, M = np.where(diag, 1.0, val.real), np.where(diag, 0.2, val.imag)
    for nsys in (2, 64):
        B = np.zeros((5000, 64), dtype=np.complex128)
        B[:, :nsys] = crandn(np.random.default_rng(1), 5000 * nsys).reshape(5000, nsys)
        args = (dev(rowptr), dev(col), dev(K), dev(M), [complex(0.1 + 0.001 * j, 0.01) for j in range(nsys)], dev(B))
        X, infos = hk.sweep_solve(*args, tol=1e-12)
        Y, _ = hk.sweep_solve(*args, tol=1e-12, shape=infos[0]["shape"])
        assert not torch.equal(X, Y) and torch.allclose(X, Y, rtol=1e-9, atol=1e-11)
