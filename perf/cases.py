"""Workloads of the complex Helmholtz Krylov path, for timing and comparison.

Each case is one call, or a short sequence of calls, that a program using
this package makes: the BLAS-1 operations of a hand-written Krylov loop, the
CSR product, whole Jacobi-preconditioned solves with each method and
precision, a frequency sweep, an uneven batch of systems, and a
differentiable solve with its adjoint.

The systems are finite-element Helmholtz matrices K - kappa M on a jittered
box of nx x ny x nz cells of edge h = 1 / max(nx, ny, nz), split into P1
tetrahedra (15 entries per row) or used as Q1 hexahedra (27), with u = 0 on
the z = 0 face by symmetric elimination, kappa = k^2 (1 + 0.01 i) and a
random complex right-hand side: the meshes of this repository's workloads.
The wave number is given as `kl` = k times the longest edge and lies in the
low band (a fraction of a wavelength to about one wavelength per box), where
a solve takes a few hundred iterations, as the paper's does on its 648,849
rows (183), and where it can be run to a residual of 1e-12 or below, so that
two solves of one system agree to many digits.  At ten nodes per wavelength
the same systems take ten thousand iterations and more, whose number and last
iterate depend on the rounding of single sums.
"""
import itertools
import math

import numpy as np
import torch

import paper_2112_11880_amd as hk
from paper_2112_11880_amd import adjoint
from paper_2112_11880_amd.hk import SWEEP_LANES

DEV = "cuda:0"
DAMP = 0.01
_ALPHA, _BETA = 0.75 - 0.5j, -0.25 + 1.25j  # exact in both precisions


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the vector operations of one step of a user's own Krylov loop (copy,
        # axpy, scale, dot, norm) on the smallest system (a 16^3 cube): five
        # calls that are all latency
        {"name": "blas1_4913", "kind": "blas1", "n": 4913},
        # the same on the paper's vectors of 9 million elements
        {"name": "blas1_9M", "kind": "blas1", "n": 9_000_000},
        # the CSR product on the 1.8-million-row box, the paper's Table 8
        {"name": "spmv_box192", "kind": "spmv", "elem": "p1", "nx": 192, "ny": 96, "nz": 96, "kl": 3.0,
         "dtype": "c128", "tuned": True, "general": False},
        # the smallest solve, on a handle with default options
        {"name": "bicgstab_cube16", "kind": "krylov", "method": "bicgstab", "elem": "p1", "nx": 16, "ny": 16,
         "nz": 16, "kl": 3.0, "tuned": False, "tol": 1e-12},
        # an ordinary solve: the 48^3 cube of the sweep and of the adjoint
        {"name": "bicgstab_cube48", "kind": "krylov", "method": "bicgstab", "elem": "p1", "nx": 48, "ny": 48,
         "nz": 48, "kl": 3.0, "tuned": True, "tol": 1e-12},
        # the largest solve, on the 1.8-million-row box
        {"name": "bicgstab_box192", "kind": "krylov", "method": "bicgstab", "elem": "p1", "nx": 192, "ny": 96,
         "nz": 96, "kl": 3.0, "tuned": True, "tol": 1e-13},
        # the paper's second method on the 27-point rows of its matrices, odd sizes
        {"name": "tfqmr_hex41", "kind": "krylov", "method": "tfqmr", "elem": "q1", "nx": 41, "ny": 37, "nz": 43,
         "kl": 3.0, "tuned": True, "tol": 1e-12},
        # the paper's third method (l = 8) on a box of 230 thousand rows
        {"name": "bicgstab8_box96", "kind": "krylov", "method": "bicgstab_l", "elem": "p1", "nx": 96, "ny": 48,
         "nz": 48, "kl": 3.0, "tuned": True, "tol": 1e-12},
        # complex64 inner iterations refined in complex128, odd sizes
        {"name": "mixed_box97", "kind": "mixed", "elem": "p1", "nx": 97, "ny": 61, "nz": 45, "kl": 2.0,
         "tuned": True, "tol": 1e-12},
        # 64 frequencies around k0 on the 48^3 cube in one call
        {"name": "sweep64_cube48", "kind": "sweep", "nx": 48, "ny": 48, "nz": 48, "kl": 2.0, "nsys": 64,
         "tol": 1e-12},
        # 32 cubes of 8 to 48 cells in one call
        {"name": "uneven32", "kind": "uneven", "nsys": 32, "least": 8, "most": 48, "kl": 2.0, "tol": 1e-12},
        # forward solve, loss at 256 nodes and both gradients, 216 speed blocks
        {"name": "adjoint_cube48", "kind": "adjoint", "cells": 48, "block": 8, "kl": 2.0, "tol": 1e-12},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _box(rng, lo, hi):
    """Three edge lengths whose product of nodes spreads over lo .. hi in its logarithm."""
    side = math.exp(rng.uniform(math.log(lo), math.log(hi)) / 3)
    a, b = rng.uniform(0.6, 1.6), rng.uniform(0.6, 1.6)
    return {"nx": max(4, round(side * a)), "ny": max(4, round(side * b)), "nz": max(4, round(side / (a * b)))}


def draw(rng):
    kind = rng.choice(["blas1", "spmv", "spmv", "krylov", "krylov", "krylov", "krylov", "mixed", "sweep",
                       "uneven", "adjoint"])
    if kind == "blas1":
        return {"kind": kind, "n": _log_int(rng, 1000, 9_000_000)}
    if kind == "spmv":
        return {"kind": kind, "elem": rng.choice(["p1", "q1"]), **_box(rng, 2000, 700_000),
                "kl": round(rng.uniform(0.5, 12.0), 2), "dtype": rng.choice(["c128", "c128", "c64"]),
                "tuned": rng.random() < 0.5, "general": rng.random() < 0.5}
    if kind == "krylov":
        return {"kind": kind, "method": rng.choice(["bicgstab", "bicgstab", "tfqmr", "bicgstab_l"]),
                "elem": rng.choice(["p1", "p1", "q1"]), **_box(rng, 2000, 500_000),
                "kl": round(rng.uniform(0.5, 3.0), 2), "tuned": rng.random() < 0.5, "tol": 1e-12}
    if kind == "mixed":
        return {"kind": kind, "elem": rng.choice(["p1", "q1"]), **_box(rng, 4000, 300_000),
                "kl": round(rng.uniform(0.5, 2.0), 2), "tuned": rng.random() < 0.5, "tol": 1e-12}
    if kind == "sweep":
        return {"kind": kind, **_box(rng, 3000, 110_000), "kl": round(rng.uniform(0.5, 2.0), 2),
                "nsys": rng.randint(3, 64), "tol": 1e-12}
    if kind == "uneven":
        return {"kind": kind, "nsys": rng.randint(2, 32), "least": rng.randint(5, 12), "most": rng.randint(16, 40),
                "kl": round(rng.uniform(0.5, 2.0), 2), "tol": 1e-12}
    return {"kind": kind, "cells": 4 * rng.randint(4, 11), "block": 4, "kl": round(rng.uniform(0.5, 2.0), 2),
            "tol": 1e-12}


# ------------------------------------------------------------------ meshes

_AXES = list(itertools.permutations(range(3)))
_CORNERS = list(itertools.product((0, 1), repeat=3))
_OFFS = {
    # couplings of the tetrahedra along the cube's (0,0,0)-(1,1,1) diagonal,
    # and of the hexahedra, in ascending order of the node number
    "p1": [o for o in itertools.product((-1, 0, 1), repeat=3) if min(o) >= 0 or max(o) <= 0],
    "q1": list(itertools.product((-1, 0, 1), repeat=3)),
}


def _tets(coords, corner, strides):
    """(local offsets, volumes, gradients) of the six tetrahedra of every cell."""
    for perm in _AXES:
        at, offs = [0, 0, 0], [(0, 0, 0)]
        for axis in perm:
            at[axis] = 1
            offs.append(tuple(at))
        lin = [sum(o * s for o, s in zip(off, strides)) for off in offs]
        X = [coords[corner + q] for q in lin]
        e1, e2, e3 = X[1] - X[0], X[2] - X[0], X[3] - X[0]
        c = [torch.cross(e2, e3, dim=1), torch.cross(e3, e1, dim=1), torch.cross(e1, e2, dim=1)]
        det = (e1 * c[0]).sum(1)
        g = [x / det[:, None] for x in c]
        yield offs, lin, det.abs() / 6, [-(g[0] + g[1] + g[2])] + g


def _mesh(nx, ny, nz, rng, jitter=0.2):
    """Node coordinates (longest edge 1), node strides, first corner of every cell, Dirichlet mask."""
    h = 1.0 / max(nx, ny, nz)
    dims = (nx + 1, ny + 1, nz + 1)
    strides = ((ny + 1) * (nz + 1), nz + 1, 1)
    ijk = torch.stack(torch.meshgrid(*[torch.arange(d, device=DEV) for d in dims], indexing="ij"), -1).reshape(-1, 3)
    d = torch.from_numpy(rng.uniform(-jitter * h, jitter * h, (ijk.shape[0], 3))).to(DEV)
    last = torch.tensor([nx, ny, nz], device=DEV)
    d[(ijk == 0) | (ijk == last)] = 0.0
    corner = torch.nonzero((ijk < last).all(1)).reshape(-1)
    return ijk * h + d, ijk, strides, corner, ijk[:, 2] == 0


def _assemble(elem, coords, corner, strides):
    """K and M as (nodes, offsets) arrays, each symmetric pair of entries added in the same step."""
    offs = _OFFS[elem]
    slot = {o: s for s, o in enumerate(offs)}
    S, n = len(offs), coords.shape[0]
    K = torch.zeros(n * S, dtype=torch.float64, device=DEV)
    M = torch.zeros_like(K)

    def add(oa, ob, la, lb, k, m):
        d = tuple(y - x for x, y in zip(oa, ob))
        at = (corner + la) * S + slot[d]
        K[at] += k
        M[at] += m
        if oa != ob:
            at = (corner + lb) * S + slot[tuple(-v for v in d)]
            K[at] += k
            M[at] += m

    if elem == "p1":
        for lo, lin, vol, G in _tets(coords, corner, strides):
            for a in range(4):
                for b in range(a, 4):
                    add(lo[a], lo[b], lin[a], lin[b], vol * (G[a] * G[b]).sum(1), vol / (10.0 if a == b else 20.0))
    else:
        lin = [sum(o * s for o, s in zip(off, strides)) for off in _CORNERS]
        X = torch.stack([coords[corner + q] for q in lin], 1)
        sg = torch.tensor(_CORNERS, dtype=torch.float64, device=DEV) * 2 - 1
        k = torch.zeros(corner.numel(), 8, 8, dtype=torch.float64, device=DEV)
        m = torch.zeros_like(k)
        for pt in itertools.product((-1 / math.sqrt(3), 1 / math.sqrt(3)), repeat=3):
            f = (1 + sg * torch.tensor(pt, dtype=torch.float64, device=DEV)) / 2
            N = f.prod(1)
            dN = torch.stack([sg[:, 0] / 2 * f[:, 1] * f[:, 2], f[:, 0] * sg[:, 1] / 2 * f[:, 2],
                              f[:, 0] * f[:, 1] * sg[:, 2] / 2], 1)
            J = (X[:, :, :, None] * dN[None, :, None, :]).sum(1)       # d x_i / d xi_j
            c = [torch.cross(J[:, :, (j + 1) % 3], J[:, :, (j + 2) % 3], dim=1) for j in range(3)]
            det = (J[:, :, 0] * c[0]).sum(1)
            inv = torch.stack(c, 1) / det[:, None, None]               # d xi_j / d x_i
            G = (dN[None, :, :, None] * inv[:, None, :, :]).sum(2)
            k += det[:, None, None] * (G[:, :, None, :] * G[:, None, :, :]).sum(-1)
            m += det[:, None, None] * (N[:, None] * N[None, :])
        for a in range(8):
            for b in range(a, 8):
                add(_CORNERS[a], _CORNERS[b], lin[a], lin[b], k[:, a, b], m[:, a, b])
    return K.reshape(n, S), M.reshape(n, S)


def _pattern(elem, ijk, strides, dirichlet):
    """Columns and kept entries, as (nodes, offsets) arrays; rows and columns of u = 0 nodes go, their diagonal stays."""
    offs = torch.tensor(_OFFS[elem], device=DEV)
    nb = ijk[:, None, :] + offs[None]
    keep = ((nb >= 0) & (nb <= ijk[-1])).all(-1)
    col = torch.arange(ijk.shape[0], device=DEV)[:, None] + (offs * torch.tensor(strides, device=DEV)).sum(1)[None]
    col = torch.where(keep, col, 0)
    keep &= ~dirichlet[:, None] & ~dirichlet[col]
    keep[:, len(_OFFS[elem]) // 2] = True
    return col, keep


def _system(elem, nx, ny, nz, seed):
    """Slot arrays of one mesh: pattern, K and M (u = 0 rows: 1 and 0 on the diagonal), and the right-hand side."""
    rng = np.random.default_rng(seed)
    coords, ijk, strides, corner, dirichlet = _mesh(nx, ny, nz, rng)
    K, M = _assemble(elem, coords, corner, strides)
    col, keep = _pattern(elem, ijk, strides, dirichlet)
    mid = K.shape[1] // 2
    K[dirichlet, mid], M[dirichlet, mid] = 1.0, 0.0
    z = torch.zeros((), dtype=torch.float64, device=DEV)
    K, M = torch.where(keep, K, z), torch.where(keep, M, z)
    b = _complex(rng, K.shape[0])
    b[dirichlet] = 0
    return {"col": torch.where(keep, col, 0), "keep": keep, "K": K, "M": M, "b": b, "dirichlet": dirichlet,
            "coords": coords, "ijk": ijk, "strides": strides, "corner": corner}


def _complex(rng, n):
    v = rng.standard_normal((2, n)) / math.sqrt(2.0)
    return torch.complex(torch.from_numpy(v[0]).to(DEV), torch.from_numpy(v[1]).to(DEV))


def _kappa(kl):
    return complex(kl * kl, DAMP * kl * kl)


def _shift(s, kappa):
    return torch.complex(s["K"] - kappa.real * s["M"], -kappa.imag * s["M"])


def _csr(s):
    rowptr = torch.zeros(s["keep"].shape[0] + 1, dtype=torch.int32, device=DEV)
    rowptr[1:] = s["keep"].sum(1).cumsum(0)
    return rowptr, s["col"][s["keep"]].to(torch.int32)


# ------------------------------------------------------------------ state

def _adjoint_lists(s, cells, block):
    """Speed blocks of block^3 cells: the mass of every entry by block, the tetrahedra by block."""
    nb = cells // block
    cell = s["ijk"][s["corner"]] // block
    blk = (cell[:, 0] * nb + cell[:, 1]) * nb + cell[:, 2]
    slot = {o: i for i, o in enumerate(_OFFS["p1"])}
    S, live = len(slot), s["keep"].reshape(-1) & ~s["dirichlet"].repeat_interleave(len(slot))
    where, val, nodes, vols = [], [], [], []
    for lo, lin, vol, _ in _tets(s["coords"], s["corner"], s["strides"]):
        nodes.append(torch.stack([s["corner"] + q for q in lin], 1))
        vols.append(vol)
        for a in range(4):
            for b in range(4):
                at = (s["corner"] + lin[a]) * S + slot[tuple(y - x for x, y in zip(lo[a], lo[b]))]
                where.append(at * nb ** 3 + blk)
                val.append(vol / (10.0 if a == b else 20.0))
    where, val = torch.cat(where), torch.cat(val)
    ok = live[where // nb ** 3]
    where, order = torch.sort(where[ok], stable=True)
    val = val[ok][order]
    key, count = torch.unique_consecutive(where, return_counts=True)
    # sums of the runs in order: a run has at most a few tens of terms
    first, got = count.cumsum(0) - count, torch.zeros(key.numel(), dtype=torch.float64, device=DEV)
    for k in range(int(count.max())):
        more = count > k
        got[more] += val[first[more] + k]
    entry = torch.cumsum(s["keep"].reshape(-1), 0) - 1
    nnz = int(entry[-1]) + 1
    ptr = torch.zeros(nnz + 1, dtype=torch.int32, device=DEV)
    ptr[1:] = torch.bincount(entry[key // nb ** 3], minlength=nnz).cumsum(0)
    nodes, vols, tblk = torch.cat(nodes), torch.cat(vols), blk.repeat(6)
    tblk, order = torch.sort(tblk, stable=True)
    tptr = torch.zeros(nb ** 3 + 1, dtype=torch.int32, device=DEV)
    tptr[1:] = torch.bincount(tblk, minlength=nb ** 3).cumsum(0)
    return {"bm_ptr": ptr, "bm_blk": (key % nb ** 3).to(torch.int32), "bm_val": got,
            "tet_nodes": nodes[order].to(torch.int32).contiguous(), "tet_ptr": tptr, "tet_vol": vols[order].contiguous(),
            "bm_slot": key // nb ** 3, "nblocks": nb ** 3}


def _uneven_parts(case, seed):
    rng = np.random.default_rng(seed)
    sizes = np.random.default_rng(2).integers(case["least"], case["most"] + 1, case["nsys"])
    sizes[0] = case["most"]
    return [_system("p1", int(v), int(v), int(v), int(rng.integers(1 << 30))) for v in sizes]


def _vectors(case, seed):
    rng = np.random.default_rng(seed)
    return [_complex(rng, case["n"]) for _ in range(2)]


def _speeds(n, seed):
    return torch.from_numpy(np.random.default_rng(seed + 7).uniform(300.0, 400.0, n)).to(DEV)


def _samples(s, seed):
    free = np.flatnonzero(~s["dirichlet"].cpu().numpy())
    return torch.from_numpy(np.sort(np.random.default_rng(seed + 5).choice(free, 256, replace=False))).to(DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "blas1":
        x, y = _vectors(case, seed)
        return {"case": case, "x": x, "y0": y, "y": torch.empty_like(y)}
    if kind == "uneven":
        parts = _uneven_parts(case, seed)
        rowptr, col, val, off = [torch.zeros(1, dtype=torch.int32, device=DEV)], [], [], [0]
        nnz = 0
        for s in parts:
            rp, c = _csr(s)
            rowptr.append(rp[1:] + nnz)
            col.append(c + off[-1])
            val.append(_shift(s, _kappa(case["kl"]))[s["keep"]])
            nnz += c.numel()
            off.append(off[-1] + s["b"].numel())
        A = hk.CSR(torch.cat(rowptr), torch.cat(col), torch.cat(val))
        return {"case": case, "A": A, "off": off, "b": torch.cat([s["b"] for s in parts])}
    if kind == "sweep":
        s = _system("p1", case["nx"], case["ny"], case["nz"], seed)
        rowptr, col = _csr(s)
        B = torch.zeros(s["b"].numel(), SWEEP_LANES, dtype=torch.complex128, device=DEV)
        B[:, : case["nsys"]] = s["b"][:, None]
        return {"case": case, "rowptr": rowptr, "col": col, "K": s["K"][s["keep"]], "M": s["M"][s["keep"]],
                "kappa": _sweep_kappas(case), "B": B}
    if kind == "adjoint":
        s = _system("p1", case["cells"], case["cells"], case["cells"], seed)
        lists = _adjoint_lists(s, case["cells"], case["block"])
        rowptr, col = _csr(s)
        prob = adjoint.HelmholtzProblem(
            rowptr=rowptr, col=col, K=s["K"][s["keep"]], dirichlet=s["dirichlet"].to(torch.uint8),
            omega=_omega(case), damp=DAMP,
            **{k: lists[k] for k in ("bm_ptr", "bm_blk", "bm_val", "tet_nodes", "tet_ptr", "tet_vol")})
        return {"case": case, "prob": prob, "g": s["b"].requires_grad_(), "S": _samples(s, seed),
                "c": _speeds(lists["nblocks"], seed).requires_grad_()}
    s = _system(case["elem"], case["nx"], case["ny"], case["nz"], seed)
    rowptr, col = _csr(s)
    val, b = _shift(s, _kappa(case["kl"]))[s["keep"]], s["b"]
    if case.get("dtype") == "c64":
        val, b = val.to(torch.complex64), b.to(torch.complex64)
    st = {"case": case, "A": hk.CSR(rowptr, col, val, autotune=case["tuned"]), "b": b}
    if kind == "spmv":
        st["y0"] = _complex(np.random.default_rng(seed + 3), b.numel()).to(b.dtype)
        st["y"] = st["y0"].clone()
    return st


def _sweep_kappas(case):
    return [_kappa(k) for k in np.linspace(0.5 * case["kl"], 1.5 * case["kl"], case["nsys"])]


def _omega(case):
    return case["kl"] * 300.0


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "blas1":
        x, y = st["x"], hk.zcopy(st["y0"], st["y"])
        hk.zaxpy(_ALPHA, x, y)
        hk.zscal(_BETA, y)
        return hk.zdotc(x, y), hk.dznrm2(y), y
    if kind == "spmv":
        if case["general"]:
            return (st["A"].spmv(st["b"], st["y0"].clone(), alpha=_ALPHA, beta=_BETA),
                    st["A"].residual(st["y0"], st["b"], st["y"]))
        return st["A"].spmv(st["b"], st["y"])
    if kind == "krylov":
        return hk.krylov_solve(st["A"], st["b"], tol=case["tol"], method=case["method"])[0]
    if kind == "mixed":
        return hk.krylov_solve_mixed(st["A"], st["b"], outer_tol=case["tol"])[0]
    if kind == "sweep":
        return hk.sweep_solve(st["rowptr"], st["col"], st["K"], st["M"], st["kappa"], st["B"], tol=case["tol"])[0]
    if kind == "uneven":
        return hk.blockdiag_solve(st["A"], st["off"], st["b"], tol=case["tol"])[0]
    u = adjoint.helmholtz_solve(st["g"], st["c"], st["prob"], tol=case["tol"])
    loss = u[st["S"]].abs().square().sum()
    grad_g, grad_c = torch.autograd.grad(loss, (st["g"], st["c"]))
    return u, grad_g, grad_c


# ------------------------------------------------------------------ work

def _size(elem, nx, ny, nz):
    """Rows and entries of a mesh's matrix."""
    n = (nx + 1) * (ny + 1) * (nz + 1)
    nnz = sum((nx + 1 - abs(a)) * (ny + 1 - abs(b)) * max(0, nz - abs(c)) for a, b, c in _OFFS[elem])
    return n, nnz + (nx + 1) * (ny + 1)


def _iterations(elem, n):
    """BiCGStab iterations to 1e-12 in the low band, about proportional to the nodes along an edge."""
    return (10.5 if elem == "p1" else 5.8) * n ** (1 / 3)


def _bicgstab(n, nnz, its, val=16, vec=16):
    """its iterations: two products (value and column of each entry) and 14 passes over vectors."""
    return its * (2 * ((val + 4) * nnz + 4 * n + 2 * vec * n) + 14 * vec * n), its * (16 * nnz + 80 * n)


def work(case):
    kind = case["kind"]
    if kind == "blas1":
        n = case["n"]
        return {"bytes": n * (32 + 16 + 48 + 32 + 32), "flops": n * (8 + 6 + 8 + 4)}
    if kind == "uneven":
        sizes = np.random.default_rng(2).integers(case["least"], case["most"] + 1, case["nsys"])
        sizes[0] = case["most"]
        parts = [_bicgstab(*_size("p1", int(v), int(v), int(v)), _iterations("p1", int(v) ** 3)) for v in sizes]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if kind == "adjoint":
        c = case["cells"]
        b, f = _bicgstab(*_size("p1", c, c, c), 2 * _iterations("p1", c ** 3))
        return {"bytes": b, "flops": f}
    n, nnz = _size(case.get("elem", "p1"), case["nx"], case["ny"], case["nz"])
    its = _iterations(case.get("elem", "p1"), n)
    if kind == "spmv":
        v = 8 if case["dtype"] == "c64" else 16
        calls = 2 if case["general"] else 1
        return {"bytes": calls * ((v + 4) * nnz + (4 + 2 * v) * n) + (calls - 1) * v * n, "flops": calls * 8 * nnz}
    if kind == "sweep":
        # 20 passes over the systems' vectors and the shared matrix twice per iteration
        return {"bytes": its * (20 * 16 * n * case["nsys"] + 2 * 20 * nnz), "flops": its * case["nsys"] * (24 * nnz + 80 * n)}
    if kind == "mixed":
        b, f = _bicgstab(n, nnz, 1.3 * its, val=8, vec=8)
        return {"bytes": b, "flops": f}
    b, f = _bicgstab(n, nnz, its)
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ 64-bit values

def _apply(col, val, x):
    """Row sums of val * x[col]."""
    y = torch.zeros_like(x)
    for s in range(col.shape[1]):
        y += val[:, s] * x[col[:, s]]
    return y


def _reference(op, diag, b):
    """Columns of x with op(x) = b: Jacobi BiCGStab in complex128, each column on its own, restarted on the true
    residual until that has stopped falling."""
    x, best, bn = torch.zeros_like(b), None, torch.linalg.vector_norm(b, dim=0)
    for _ in range(4):
        r = b - op(x)
        rn = (torch.linalg.vector_norm(r, dim=0) / bn).max().item()
        if best is not None and not rn < 0.25 * best[0]:
            break
        best = (rn, x.clone())
        x = x + _bicgstab_columns(op, diag, r)
    r = b - op(x)
    rn = (torch.linalg.vector_norm(r, dim=0) / bn).max().item()
    return x if rn < best[0] else best[1]


def _bicgstab_columns(op, diag, b, tol=1e-11, most=6000):
    dot = lambda u, v: (u.conj() * v).sum(0)  # noqa: E731
    x = torch.zeros_like(b)
    r, rh = b.clone(), b
    p = r.clone()
    rho, bn2 = dot(rh, r), dot(b, b).real
    live = bn2 > 0
    one = torch.ones_like(rho)
    for it in range(most):
        ph = p / diag
        v = op(ph)
        al = torch.where(live, rho / torch.where(live, dot(rh, v), one), 0 * one)
        s = r - al * v
        sh = s / diag
        t = op(sh)
        tt = dot(t, t)
        om = torch.where(live, dot(t, s) / torch.where(live, tt, one), 0 * one)
        x = x + al * ph + om * sh
        r = torch.where(live, s - om * t, r)
        live = live & (dot(r, r).real > tol * tol * bn2)
        if it % 16 == 15 and not bool(live.any()):
            break
        new = dot(rh, r)
        be = torch.where(live, new / torch.where(live, rho, one) * (al / torch.where(live, om, one)), 0 * one)
        rho = torch.where(live, new, rho)
        p = torch.where(live, r + be * (p - om * v), p)
    return x


def _solve_slots(s, val, b):
    mid = s["col"].shape[1] // 2
    return _reference(lambda x: _apply(s["col"], val, x), val[:, mid], b)


def exact(case, seed):
    kind = case["kind"]
    if kind == "blas1":
        x, y = _vectors(case, seed)
        y = _BETA * (y + _ALPHA * x)
        return (x.conj() * y).sum().reshape(1), torch.linalg.vector_norm(y).reshape(1), y
    if kind == "uneven":
        out = [_solve_slots(s, _shift(s, _kappa(case["kl"])), s["b"]) for s in _uneven_parts(case, seed)]
        return torch.cat(out)
    if kind == "sweep":
        s = _system("p1", case["nx"], case["ny"], case["nz"], seed)
        mid = s["col"].shape[1] // 2
        kap = torch.tensor(_sweep_kappas(case), dtype=torch.complex128, device=DEV)
        Kc, Mc = s["K"].to(torch.complex128), s["M"].to(torch.complex128)

        def op(x):
            y = torch.zeros_like(x)
            for q in range(s["col"].shape[1]):
                y += (Kc[:, q, None] - kap[None] * Mc[:, q, None]) * x[s["col"][:, q]]
            return y

        X = torch.zeros(s["b"].numel(), SWEEP_LANES, dtype=torch.complex128, device=DEV)
        X[:, : case["nsys"]] = _reference(op, Kc[:, mid, None] - kap[None] * Mc[:, mid, None],
                                          s["b"][:, None].expand(-1, case["nsys"]).contiguous())
        return X
    if kind == "adjoint":
        s = _system("p1", case["cells"], case["cells"], case["cells"], seed)
        L = _adjoint_lists(s, case["cells"], case["block"])
        c, S = _speeds(L["nblocks"], seed), _samples(s, seed)
        w = complex(1.0, DAMP) * _omega(case) ** 2
        blk, slots = L["bm_blk"].long(), s["K"].numel()
        mass = torch.zeros(slots, dtype=torch.float64, device=DEV)
        mass.index_add_(0, L["bm_slot"], L["bm_val"] / c[blk] ** 2)
        mass = mass.reshape(s["K"].shape)
        val = torch.complex(s["K"] - w.real * mass, -w.imag * mass)
        u = _solve_slots(s, val, s["b"])
        gu = torch.zeros_like(u)
        gu[S] = 2 * u[S]
        lam = _solve_slots(s, val, gu.conj().resolve_conj())
        # every entry's mass by block: lambda^T M_b u summed over the entries of the block
        node, to = L["bm_slot"] // s["K"].shape[1], s["col"].reshape(-1)[L["bm_slot"]]
        q = torch.zeros(L["nblocks"], dtype=torch.complex128, device=DEV)
        q.index_add_(0, blk, L["bm_val"] * lam[node] * u[to])
        return u, lam.conj().resolve_conj(), -(2 * w * q / c ** 3).real
    s = _system(case["elem"], case["nx"], case["ny"], case["nz"], seed)
    val, b = _shift(s, _kappa(case["kl"])), s["b"]
    if kind == "spmv":
        if case["dtype"] == "c64":
            val, b = val.to(torch.complex64).to(torch.complex128), b.to(torch.complex64).to(torch.complex128)
        y = _apply(s["col"], val, b)
        if not case["general"]:
            return y
        y0 = _complex(np.random.default_rng(seed + 3), b.numel())
        if case["dtype"] == "c64":
            y0 = y0.to(torch.complex64).to(torch.complex128)
        return _ALPHA * y + _BETA * y0, y0 - y
    return _solve_slots(s, val, b)
