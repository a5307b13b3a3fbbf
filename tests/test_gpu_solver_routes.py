"""The solves' several routes (resident launches, sliced products, kernels per
phase) held against each other: rounding, exits, fallbacks, what is reported."""
import numpy as np
import pytest

from synth import helmholtz as H
from synth import hexahedra as HX

from test_gpu_resident import block_diagonal as dominant_blocks
from test_gpu_resident import dominant

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


def mesh_system(cells, elem="p1", seed=3, kappa=complex(4.0, 0.04)):
    m = H.make_mesh(*cells, 1.0 / max(cells), jitter=0.2, rng=np.random.default_rng(seed))
    p = H.build_problem(m) if elem == "p1" else HX.build_hex_problem(m)
    return p.rowptr, p.col, H.helmholtz_values(p, kappa), H.complex_rhs(np.random.default_rng(seed), p.n, p.dirichlet)


def with_far_entries(rowptr, col, val, distance, size):
    """One more entry, at the given distance, in every row that reaches so far."""
    n = rowptr.shape[0] - 1
    rows = np.concatenate([np.repeat(np.arange(n), np.diff(rowptr)), np.arange(n - distance)])
    cols = np.concatenate([col, np.arange(n - distance) + distance])
    vals = np.concatenate([val, np.full(n - distance, size)])
    order = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return rp, cols[order].astype(np.int32), vals[order]


@pytest.mark.parametrize("elem,far,first", [("p1", 0, 1), ("q1", 0, 1), ("q1", 9000, 2)])
def test_row_sums_round_no_more_than_row_blocks(hk, elem, far, first):
    """The rounding of the products is what the true residual of a BiCGStab(8)
    solve to 1e-12 is left with: some thousand of them, so that it follows their
    size within a few percent.  On a random vector the row blocks of 32 rows
    round by 1.68e-16 (rows of 15 entries) and 1.95e-16 (27), the resident rows by
    1.52e-16 and 1.71e-16, the slices of 27 by 1.73e-16, one chain of multiply-adds
    by 2.7e-16 and 3.5e-16: ratios of 0.9 here, of 1.6 and 1.8 with one chain."""
    rowptr, col, val, b = mesh_system((30, 29, 30), elem)
    if far:  # 28 entries: not resident, products on slices
        rowptr, col, val = with_far_entries(rowptr, col, val, far, 1e-9 * abs(val).max())
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    B = hk.CSR(A.rowptr, A.col, A.val)
    B.set_plan(64, 32)
    print("[case] rounding of the row sums", elem, far, flush=True)
    _, here = hk.krylov_solve(A, dev(b), tol=1e-12, method="bicgstab_l", ell=8)
    _, blocks = hk.krylov_solve(B, dev(b), tol=1e-12, method="bicgstab_l", ell=8)
    assert here["status"] == blocks["status"] == hk.HK_OK
    assert here["shape"][0] == first and blocks["shape"][:2] == [64, 32], (here, blocks)
    assert here["relres_true"] <= 1.15 * blocks["relres_true"], (here, blocks)


@pytest.mark.parametrize("cells,l8", [((31, 31, 31), 1), ((32, 31, 31), 64), ((60, 45, 50), 64), ((76, 60, 58), 64)])
def test_bicgstab_8_keeps_the_order_of_its_sums(hk, cells, l8):
    """Above 32,768 rows BiCGStab(8) to less than 1e-10 gives the bits of the
    kernels per phase in the handle's own shape, whether the system would fit the
    registers (143,106 rows) or have its products on slices (277,123); a looser
    tolerance and l = 4 take the faster routes."""
    rowptr, col, val, b = mesh_system(cells)
    n = b.shape[0]
    print("[case] order of sums", n, flush=True)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    other = 1 if n <= 262144 else 2
    kw = dict(method="bicgstab_l", max_iter=4)
    for ell, tol, first in ((4, 1e-12, other), (8, 1e-10, other), (8, 1e-12, l8), (8, 0.0, l8)):
        x, info = hk.krylov_solve(A, dev(b), tol=tol, ell=ell, **kw)
        assert info["shape"][0] == first, (ell, tol, info)
    B = hk.CSR(A.rowptr, A.col, A.val)
    p = A.plan()
    B.set_plan(p["lanes_per_row"], p["rows_per_group"], p["grid"])
    kw["max_iter"] = 400
    x, info = hk.krylov_solve(A, dev(b), tol=1e-12, **kw)
    y, _ = hk.krylov_solve(B, dev(b), tol=1e-12, **kw)
    assert info["status"] == hk.HK_OK
    assert torch.equal(x, y) == (l8 == 64)
    assert torch.linalg.vector_norm(x - y) <= 1e-9 * torch.linalg.vector_norm(y)
    T = hk.CSR(A.rowptr, A.col, A.val, autotune=True)
    for method, tol in (("bicgstab", 1e-3), ("bicgstab_l", 1e-12)):  # the first may tune and keep slices
        _, info = hk.krylov_solve(T, dev(b), tol=tol, method=method)
    assert (info["shape"][0] == 1) if l8 == 1 else (info["shape"][0] not in (1, 2) and info["shape_tuned"]), info


@pytest.mark.parametrize("method,kw", [("bicgstab", {}), ("tfqmr", {}), ("bicgstab_l", {"ell": 2}), ("bicgstab_l", {"ell": 8})])
@pytest.mark.parametrize("cells,elem", [((20, 19, 19), "p1"), ((20, 19, 19), "q1"), ((25, 23, 24), "p1"), ((25, 23, 24), "q1")])
def test_packed_launch_has_room(hk, oracle, method, kw, cells, elem):
    """8,400 and 15,600 rows: 33 and 61 workgroups of 256 threads on one XCD, two of
    them on some of its 32 CUs.  Every method runs resident there."""
    rowptr, col, val, b = mesh_system(cells, elem)
    print("[case] packed", method, kw, b.shape[0], elem, flush=True)
    x, info = hk.krylov_solve(hk.CSR(dev(rowptr), dev(col), dev(val)), dev(b), tol=1e-9, method=method, **kw)
    assert info["status"] == hk.HK_OK and info["shape"] == [1, 1, 4, 0], info
    r = oracle.residual(rowptr, col, val, b, x.cpu().numpy())
    assert np.linalg.norm(r) <= 1.05e-9 * np.linalg.norm(b)


def block_diagonal(parts):
    """One matrix of several systems (rowptr, col, val, b) and their row offsets."""
    off = np.concatenate([[0], np.cumsum([p[3].shape[0] for p in parts])])
    nnz = np.cumsum([0] + [p[1].shape[0] for p in parts])
    rowptr = np.concatenate([[0]] + [p[0][1:] + z for p, z in zip(parts, nnz)]).astype(np.int32)
    col = np.concatenate([p[1] + o for p, o in zip(parts, off)]).astype(np.int32)
    return off, rowptr, col, np.concatenate([p[2] for p in parts]), np.concatenate([p[3] for p in parts])


def test_batch_waits_for_earlier_systems(hk, monkeypatch):
    """Systems of 99, 97, 89 and 61 workgroups (27 entries: one row per thread) on 256:
    the second one never converges, and most workgroups of the fourth are free from
    the start while eight of them solve the second, for some 0.2 s.  A barrier limit of
    40 ms does not end that wait: the bits are those under the default limit, which the
    tiled launch does not give."""
    easy = [mesh_system(c, "q1", seed=k, kappa=complex(1.0, 0.01)) for k, c in enumerate([(36, 36, 36), (34, 35, 35), (30, 31, 30)])]
    hard = mesh_system((36, 36, 35), "q1", seed=7, kappa=complex(500.0, 5.0))
    off, rowptr, col, val, b = block_diagonal([easy[0], hard, easy[1], easy[2]])
    assert [-(-(int(hi) - int(lo)) // 512) for lo, hi in zip(off, off[1:])] == [99, 97, 89, 61]
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    kw = dict(tol=1e-25, max_iter=20000)
    print("[case] batch, default barrier limit", flush=True)
    x, infos = hk.blockdiag_solve(A, off, dev(b), **kw)
    assert infos[1]["iters"] > 8000 and all(infos[k]["status"] == hk.HK_OK and infos[k]["iters"] < 2000 for k in (0, 2, 3)), infos
    print("[case] batch, 40 ms", flush=True)
    monkeypatch.setenv("HK_BARRIER_SPIN_TICKS", "4000000")
    y, late = hk.blockdiag_solve(A, off, dev(b), **kw)
    assert torch.equal(x, y) and [i["iters"] for i in late] == [i["iters"] for i in infos]
    z, _ = hk.blockdiag_solve(A, off, dev(b), shape=infos[0]["shape"], **kw)
    assert not torch.equal(x, z)


@pytest.mark.parametrize("sizes,row,rows_per_thread", [
    ([1], 1, (1,)), ([1, 2, 63, 64, 65, 130], 8, (1, 2)), ([700, 5, 20000, 513, 1], 15, (1, 2)),
    ([40000, 70000, 3000] + [65] * 61, 15, (1, 2)), ([131073, 900, 131072, 17], 15, (2,)), ([131073, 900, 131072, 17], 8, (2,)),
    ([500, 9000, 27], 27, (1,)), ([300, 40], 28, (0,)), ([131073, 50], 27, (0,))])
def test_batch_reports_its_launch(hk, sizes, row, rows_per_thread):
    """Every form of the batch's resident launch runs where its systems fit (a refused
    launch would leave the tiled one, and 0 here)."""
    _, off, rowptr, col, val, b = dominant_blocks(sizes, row, 17)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    print("[case] batch launch", sizes[:4], row, flush=True)
    x, infos = hk.blockdiag_solve(A, off, dev(b), tol=0.0, max_iter=2)
    assert all(i["resident"] in rows_per_thread for i in infos) and len({i["resident"] for i in infos}) == 1, infos
    y, infos = hk.blockdiag_solve(A, off, dev(b), tol=0.0, max_iter=2, shape=infos[0]["shape"])
    assert all(i["resident"] == 0 for i in infos)
    assert torch.allclose(x, y, rtol=1e-9, atol=1e-10)


@pytest.mark.parametrize("n,row,nsys,rows_per_thread", [
    (512, 15, 3, (0,)), (513, 15, 3, (1, 2)), (1000, 8, 64, (1, 2)), (9000, 15, 33, (1, 2)), (20011, 15, 5, (1, 2)),
    (70001, 15, 7, (1, 2)), (131073, 15, 3, (2,)), (140000, 8, 2, (2,)), (40000, 27, 5, (1,)), (131073, 27, 2, (0,)),
    (3000, 28, 3, (0,)), (60001, 15, 4, (1, 2)), (40001, 15, 64, (1, 2)), (131072, 15, 2, (1, 2)), (100003, 15, 19, (1, 2)),
    (33000, 8, 13, (1, 2))])
def test_sweep_reports_its_launch(hk, n, row, nsys, rows_per_thread):
    """The same for the sweep: one and two rows per thread, one and several systems at a time."""
    rowptr, col, val, _ = dominant(n, row, n + row)
    diag = col == np.repeat(np.arange(n), np.diff(rowptr))
    K, M = np.where(diag, 1.0, val.real), np.where(diag, 0.2, val.imag)
    B = np.zeros((n, 64), dtype=np.complex128)
    B[:, :nsys] = np.random.default_rng(n).standard_normal((n, nsys))
    args = (dev(rowptr), dev(col), dev(K), dev(M), [complex(0.1 + 0.4 * j / nsys, 0.01 * (j + 1)) for j in range(nsys)], dev(B))
    print("[case] sweep launch", n, row, nsys, flush=True)
    X, infos = hk.sweep_solve(*args, tol=1e-14, max_iter=2)
    assert all(i["resident"] in rows_per_thread for i in infos) and len({i["resident"] for i in infos}) == 1, infos
    Y, infos = hk.sweep_solve(*args, tol=1e-14, max_iter=2, shape=infos[0]["shape"])
    assert all(i["resident"] == 0 for i in infos)
    assert torch.allclose(X, Y, rtol=1e-9, atol=1e-10)


def test_single_solves_report_their_launch(hk):
    for n, row, here in ((5000, 15, 1), (140000, 15, 2), (5000, 28, 0)):
        rowptr, col, val, b = dominant(n, row, n)
        A = hk.CSR(dev(rowptr), dev(col), dev(val))
        for method in ("bicgstab", "tfqmr", "bicgstab_l"):
            print("[case] launch", method, n, row, flush=True)
            assert hk.krylov_solve(A, dev(b), tol=1e-6, method=method)[1]["resident"] == here, (n, row, method)
        assert hk.krylov_solve_mixed(A, dev(b), outer_tol=1e-8)[1]["resident"] == here, (n, row, "mixed")


@pytest.mark.parametrize("n,nsys", [(5000, 2), (5000, 64)])
def test_batched_time_out_in_a_resident_launch(hk, monkeypatch, n, nsys):
    """With a limit of one tick the resident launch ends through its abort path, and
    so does the launch that starts over; the next calls are resident again and
    give the bits from before."""
    rowptr, col, val, _ = dominant(n, 15, 9)
    diag = col == np.repeat(np.arange(n), np.diff(rowptr))
    K, M = np.where(diag, 1.0, val.real), np.where(diag, 0.2, val.imag)
    B = np.zeros((n, 64), dtype=np.complex128)
    B[:, :nsys] = np.random.default_rng(1).standard_normal((n, nsys))
    args = (dev(rowptr), dev(col), dev(K), dev(M), [complex(0.1 + 0.001 * j, 0.01) for j in range(nsys)], dev(B))
    _, off, rp, c, v, b = dominant_blocks([3000, 900, 20000], 15, 5)
    A = hk.CSR(dev(rp), dev(c), dev(v))
    X, _ = hk.sweep_solve(*args, tol=1e-12)
    x, _ = hk.blockdiag_solve(A, off, dev(b), tol=1e-12)
    monkeypatch.setenv("HK_BARRIER_SPIN_TICKS", "1")
    print("[case] limit of one tick: sweep, batch", n, nsys, flush=True)
    with pytest.raises(hk.HKError, match="timed out"):
        hk.sweep_solve(*args, tol=1e-12)
    with pytest.raises(hk.HKError, match="timed out"):
        hk.blockdiag_solve(A, off, dev(b), tol=1e-12)
    monkeypatch.delenv("HK_BARRIER_SPIN_TICKS")
    Y, infos = hk.sweep_solve(*args, tol=1e-12)
    assert all(i["resident"] for i in infos) and torch.equal(X, Y)
    y, infos = hk.blockdiag_solve(A, off, dev(b), tol=1e-12)
    assert all(i["resident"] for i in infos) and torch.equal(x, y)


METHODS = [("bicgstab", {}), ("tfqmr", {}), ("bicgstab_l", {"ell": 4})]


@pytest.mark.parametrize("method,kw", METHODS)
@pytest.mark.parametrize("route", [64, 16, 2])
def test_kernels_per_phase_replay_graphs(hk, monkeypatch, method, kw, route):
    """The recorded chunks of the kernels per phase, on row blocks, lane groups and
    slices, give the bits of direct launches, with a chunk of 3 iterations and with
    the default one."""
    rowptr, col, val, b = mesh_system((30, 29, 30) if route == 2 else (7, 6, 6), "q1")
    if route == 2:  # 28 entries at few distances: slices
        rowptr, col, val = with_far_entries(rowptr, col, val, 9000, 1e-9 * abs(val).max())
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    if route != 2:
        A.set_plan(route, 2 if route == 16 else 32)
    for every in (3, 0):
        got = []
        for graphs in ("1", "0"):
            monkeypatch.setenv("HK_SOLVE_GRAPHS", graphs)
            print("[case] graph replay", method, route, every, graphs, flush=True)
            got.append(hk.krylov_solve(A, dev(b), tol=1e-10, check_every=every, method=method, **kw))
        (x, info), (y, direct) = got
        assert info["status"] == hk.HK_OK and info["resident"] == 0 and info["shape"][0] == route, info
        assert info == direct and torch.equal(x, y)


@pytest.mark.parametrize("method,kw", METHODS)
@pytest.mark.parametrize("plan", [None, (64, 32), (16, 2)])
def test_exits_on_every_route(hk, oracle, method, kw, plan):
    """Breakdowns, non-finite and zero right-hand sides, an exact start, the cap and a
    diagonal system, resident (no plan) and by the kernels per phase."""
    def handle(rowptr, col, val):
        A = hk.CSR(dev(np.asarray(rowptr, dtype=np.int32)), dev(np.asarray(col, dtype=np.int32)),
                   dev(np.asarray(val, dtype=np.complex128)))
        if plan:
            A.set_plan(*plan)
        return A

    def solve(A, b, **more):
        x, info = hk.krylov_solve(A, dev(np.asarray(b, dtype=np.complex128)), method=method, **kw, **more)
        assert info["resident"] == (0 if plan else 1), info
        return x.cpu().numpy(), info

    print("[case] exits", method, plan, flush=True)
    x, info = solve(handle([0, 2, 4], [0, 1, 0, 1], [1.0, -1.25, -1.25, 1.0]), [1.0, 2.0], tol=1e-12)
    assert info["status"] == hk.HK_BREAKDOWN and hk.BD_NAMES[info["breakdown"]] == "sigma"
    assert info["iters"] == 0 and np.all(x == 0)
    if method == "bicgstab":
        x, info = solve(handle([0, 3, 6, 9], list(range(3)) * 3, [1, 1, 0, 1, 1, -1, 1, -1, 1]), [1.0, 0, 0], tol=1e-14)
        assert info["status"] == hk.HK_BREAKDOWN and hk.BD_NAMES[info["breakdown"]] == "omega"
        assert info["iters"] == 1 and np.array_equal(x, np.array([1.0, 0, 0]))
    with pytest.raises(hk.HKError, match="zero diagonal"):
        solve(handle([0, 1, 2], [1, 0], [1.0, 1.0]), [1.0, 1.0])
    rng = np.random.default_rng(2)
    d, b = rng.standard_normal(40) + 3.0 + 1j * rng.standard_normal(40), rng.standard_normal(40) + 0j
    x, info = solve(handle(np.arange(41), np.arange(40), d), b, tol=1e-12)
    assert info["status"] == hk.HK_OK and info["iters"] == 1 and np.allclose(x, b / d, rtol=1e-14, atol=0)
    rowptr, col, val, b = mesh_system((9, 8, 8))
    A = handle(rowptr, col, val)
    x, info = solve(A, np.zeros_like(b))
    assert info["status"] == hk.HK_OK and info["iters"] == 0 and np.all(x == 0)
    for bad in (np.nan, np.inf):
        g = b.copy()
        g[7] = bad
        assert solve(A, g)[1]["status"] == hk.HK_NONFINITE
    xo, _ = oracle.bicgstab(rowptr, col, val, b, tol=1e-12)
    x, info = solve(A, b, x=dev(xo), tol=1e-8)
    assert info["status"] == hk.HK_OK and info["iters"] == 0
    x, info = solve(A, b, max_iter=2, tol=1e-14)
    ref = getattr(oracle, method)(rowptr, col, val, b, tol=1e-14, maxit=2, **kw)[0]
    assert info["status"] == hk.HK_NOT_CONVERGED and info["iters"] == 2
    assert np.linalg.norm(x - ref) <= 1e-10 * np.linalg.norm(ref)
    x, info, hist = hk.krylov_solve(A, dev(b), tol=1e-9, method=method, history=True, **kw)
    h = hist.cpu().numpy()
    assert info["status"] == hk.HK_OK and h.shape[0] == info["iters"] + 1
    assert h[0] == pytest.approx(1.0) and h[-1] <= 1.0001e-9 and h[-1] == pytest.approx(info["relres_rec"])


@pytest.mark.parametrize("n", [5000, 20000])
def test_bicgstab_l_starts_over_after_a_time_out(hk, oracle, monkeypatch, n):
    """A resident BiCGStab(l) whose barrier waits may take no time ends through its
    abort path, and the kernels per phase solve from the caller's start."""
    rowptr, col, val, b = dominant(n, 15, 9)
    rng = np.random.default_rng(1)
    x0 = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    monkeypatch.setenv("HK_BARRIER_SPIN_TICKS", "1")
    print("[case] bicgstab_l, limit of one tick", n, flush=True)
    x, info = hk.krylov_solve(hk.CSR(dev(rowptr), dev(col), dev(val)), dev(b), x=dev(x0), tol=1e-12, method="bicgstab_l", ell=2)
    assert info["status"] == hk.HK_OK and info["resident"] == 0, info
    r = oracle.residual(rowptr, col, val, b, x.cpu().numpy())
    assert np.linalg.norm(r) <= 1.05e-12 * np.linalg.norm(b)


def test_solves_of_two_threads_at_once(hk):
    """Two handles, each in a thread and on a stream of its own: resident launches that
    would each fill the device, with a BLAS-1 loop beside them on a third stream, give
    the bits of single calls, every time."""
    import threading
    systems = [mesh_system((44, 45, 46), seed=1), mesh_system((46, 44, 43), seed=2)]
    alone = []
    for rowptr, col, val, b in systems:
        A = hk.CSR(dev(rowptr), dev(col), dev(val))
        x, info = hk.krylov_solve(A, dev(b), tol=1e-9)
        assert info["resident"] == 1
        alone.append((A, dev(b), x, info["iters"]))
    torch.cuda.synchronize()
    got, done = [[], []], threading.Event()

    def work(k):
        A, b, _, _ = alone[k]
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(6):
                print("[case] thread", k, flush=True)
                x, info = hk.krylov_solve(A, b, tol=1e-9)
                got[k].append((x, info))
            torch.cuda.current_stream().synchronize()

    def noise():
        with torch.cuda.stream(torch.cuda.Stream()):
            u, v = torch.ones(1 << 20, dtype=torch.complex128, device=DEV), torch.zeros(1 << 20, dtype=torch.complex128, device=DEV)
            while not done.is_set():
                for _ in range(20):
                    hk.zaxpy(0.5, u, v)
                torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    beside = threading.Thread(target=noise)
    for t in [beside, *threads]:
        t.start()
    for t in threads:
        t.join()
    done.set()
    beside.join()
    for k in range(2):
        assert len(got[k]) == 6
        for x, info in got[k]:
            assert info["resident"] == 1 and info["iters"] == alone[k][3] and torch.equal(x, alone[k][2]), (k, info)


@pytest.mark.parametrize("cells,shape", [((16, 15, 16), [1, 1, 4, 0]), ((25, 23, 24), [1, 1, 4, 0]), ((48, 48, 48), [1, 1, 8, 0]),
                                         ((60, 45, 50), [1, 2, 8, 0])])
def test_resident_bicgstab_8_repeats_its_bits(hk, cells, shape):
    """l = 8 on one XCD with one and two workgroups per CU, on most CUs with one row
    per thread and with two: the same bits from call to call and from a new handle."""
    rowptr, col, val, b = mesh_system(cells)
    print("[case] repeat bicgstab(8)", b.shape[0], flush=True)
    A = hk.CSR(dev(rowptr), dev(col), dev(val))
    x, info = hk.krylov_solve(A, dev(b), tol=1e-9, method="bicgstab_l", ell=8)
    assert info["status"] == hk.HK_OK and info["shape"] == shape, info
    for again in (A, A, hk.CSR(A.rowptr, A.col, A.val)):
        y, other = hk.krylov_solve(again, dev(b), tol=1e-9, method="bicgstab_l", ell=8)
        assert other == info and torch.equal(x, y)


@pytest.mark.parametrize("n,nsys", [(5000, 3), (9000, 33), (40001, 20)])
def test_sweep_keeps_nonfinite_columns_apart(hk, n, nsys):
    """A NaN and an infinity in two right-hand sides end these systems only: the others
    have the bits that they have beside zero columns."""
    rowptr, col, val, _ = dominant(n, 15, n)
    diag = col == np.repeat(np.arange(n), np.diff(rowptr))
    K, M = np.where(diag, 1.0, val.real), np.where(diag, 0.2, val.imag)
    kap = [complex(0.1 + 0.4 * j / nsys, 0.01 * (j + 1)) for j in range(nsys)]
    B = np.zeros((n, 64), dtype=np.complex128)
    B[:, :nsys] = np.random.default_rng(n).standard_normal((n, nsys))
    B[:, [0, nsys - 1]] = 0
    bad = B.copy()
    bad[n // 2, 0], bad[1, nsys - 1] = np.nan, np.inf
    arrays = (dev(rowptr), dev(col), dev(K), dev(M), kap)
    print("[case] sweep, non-finite columns", n, nsys, flush=True)
    X, infos = hk.sweep_solve(*arrays, dev(B), tol=1e-10)
    Y, late = hk.sweep_solve(*arrays, dev(bad), tol=1e-10)
    assert all(i["resident"] for i in infos + late)
    assert [late[k]["status"] for k in (0, nsys - 1)] == [hk.HK_NONFINITE] * 2
    for k in range(1, nsys - 1):
        assert late[k]["status"] == hk.HK_OK and late[k]["iters"] == infos[k]["iters"]
    assert torch.equal(X[:, 1:nsys - 1], Y[:, 1:nsys - 1])


def outcomes(hk, monkeypatch, call, low, high, step):
    """What call() reports as the workspace limit grows from `low` to `high` bytes: -1 (refused) or its number."""
    got, limit = [], float(low)
    while limit < high:
        monkeypatch.setenv("HK_WORKSPACE_LIMIT", str(int(limit)))
        try:
            got.append(call())
        except hk.HKError as e:
            assert e.code == -3, e  # HK_ENOMEM
            got.append(-1)
        limit *= step
    monkeypatch.delenv("HK_WORKSPACE_LIMIT")
    return got


def test_small_workspaces_take_the_lean_launches(hk, monkeypatch):
    """Where a workspace with room for the resident launch or for the slices is refused
    and one without is not, the solve runs without them and to the same solution."""
    rowptr, col, val, b = dominant(5000, 15, 9)
    arrays, bd = (dev(rowptr), dev(col), dev(val)), dev(b)
    far = with_far_entries(*mesh_system((30, 29, 30), "q1")[:3], 9000, 1e-3)
    bf, farrays = dev(mesh_system((30, 29, 30), "q1")[3]), tuple(dev(a) for a in far)
    _, off, rp, c, v, bb = dominant_blocks([3000, 900, 20000], 15, 5)
    barrays, bbd = (dev(rp), dev(c), dev(v)), dev(bb)
    diag = col == np.repeat(np.arange(5000), np.diff(rowptr))
    srp, scol, sval, _ = dominant(1000, 8, 3)
    sdiag = scol == np.repeat(np.arange(1000), np.diff(srp))
    B = np.zeros((1000, 64), dtype=np.complex128)
    B[:] = np.random.default_rng(1).standard_normal((1000, 64))
    sweep = (dev(srp), dev(scol), dev(np.where(sdiag, 1.0, sval.real)), dev(np.where(sdiag, 0.2, sval.imag)),
             [complex(0.1 + 0.001 * j, 0.01) for j in range(64)], dev(B))
    assert diag.any()
    kept = {}

    def single(arrays, b, first, autotune=False, **kw):
        x, info = hk.krylov_solve(hk.CSR(*arrays, autotune=autotune), b, tol=1e-10, **kw)
        y = kept.setdefault((first, autotune, str(kw)), x)
        assert info["status"] == hk.HK_OK and torch.allclose(x, y, rtol=1e-6, atol=1e-8 * float(y.abs().max()))
        return int(info["shape"][0] == first)

    def mixed():
        x, info = hk.krylov_solve_mixed(hk.CSR(*arrays), bd, outer_tol=1e-9)
        assert info["status"] == hk.HK_OK
        return int(info["shape"][0] == 1)

    def batch():
        x, infos = hk.blockdiag_solve(hk.CSR(*barrays), off, bbd, tol=1e-10)
        assert all(i["status"] == hk.HK_OK for i in infos)
        y = kept.setdefault("batch", x)
        assert torch.allclose(x, y, rtol=1e-6, atol=1e-8)
        return infos[0]["resident"]

    def sweeps():
        X, infos = hk.sweep_solve(*sweep, tol=1e-10)
        assert all(i["status"] == hk.HK_OK for i in infos)
        Y = kept.setdefault("sweep", X)
        assert torch.allclose(X, Y, rtol=1e-6, atol=1e-8)
        return infos[0]["resident"]

    cases = [(f"{m}", lambda m=m, kw=kw: single(arrays, bd, 1, method=m, **kw), 4e5, 2e7, 1.1) for m, kw in METHODS]
    cases += [("slices", lambda: single(farrays, bf, 2), 6e6, 3e7, 1.02), ("slices, tuned", lambda: single(farrays, bf, 2, True), 6e6, 3e7, 1.02),
              ("mixed", mixed, 4e5, 2e7, 1.1), ("batch", batch, 1e6, 6e7, 1.1), ("sweep", sweeps, 1e6, 4e8, 1.3)]
    for name, call, low, high, step in cases:
        print("[case] workspace limits", name, flush=True)
        got = outcomes(hk, monkeypatch, call, low, high, step)
        if name == "slices, tuned":  # each handle's tuner may prefer another shape
            first = next(k for k, g in enumerate(got) if g >= 0)
            assert first > 0 and -1 not in got[first:], (name, got)
        else:
            assert got == sorted(got) and {-1, 0}.issubset(got) and got[-1] >= 1, (name, got)
