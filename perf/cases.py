"""Performance cases: calls a program makes through the package's public entry
points (symbolic, batch, symbolic_noalloc, Server), from a 40 x 40 grid to the
64^3 27-point and 1000^2 9-point stencils of bench.py.

listed() names the fixed cases, draw() gives more of the same ranges,
prepare() makes what a program holds before the call (the matrices, output
arrays, an open server), run() is one pass and returns its whole outputs.
Matrices are this repository's stencils. Grid and dropped entries belong to the
case, so that every seed has factors of the same size; the seed places a few rows
that are coupled to nothing (a diagonal entry only) among the others, which moves
every other row and column.
"""
from __future__ import annotations

import functools
import math
import weakref

import numpy as np
import torch

import paper_2007_00840_amd as g
import synth


def _one(name, kind, dims, nd=True, host=False, l_csr=False, supernodes=True, max_supernode=0, mode="symbolic"):
    nx, ny, nz = dims
    c = {"mode": mode, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "nd": nd, "host": host, "l_csr": l_csr,
         "supernodes": supernodes, "max_supernode": max_supernode}
    if name:
        c["name"] = name
    return c


def _many(name, mode, count, n_lo, n_hi, host):
    c = {"mode": mode, "count": count, "n_lo": n_lo, "n_hi": n_hi, "host": host}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: latency of one small device-resident matrix, natural order
        _one("grid40_5pt", 5, (40, 40, 1), nd=False),
        # one small matrix handed over and returned as host arrays
        _one("host_2000_9pt", 9, (44, 45, 1), host=True),
        # results written into caller-owned device arrays, no device allocation
        _one("noalloc_100sq_9pt", 9, (100, 100, 1), mode="noalloc"),
        # odd 3D grid, L wanted row-wise, no supernode partition
        _one("lcsr_29x31x23_7pt", 7, (29, 31, 23), l_csr=True, supernodes=False),
        # mid-size 3D stencil on the device, supernodes limited to 32 rows
        _one("sn32_31x30x32_27pt", 27, (31, 30, 32), max_supernode=32),
        # a 10^5-row 2D matrix from and to host memory
        _one("host_317x315_9pt", 9, (317, 315, 1), host=True),
        # a 10^5-row 3D matrix from and to host memory (420 MB of result)
        _one("host_48cube_27pt", 27, (48, 48, 48), host=True),
        # the two large matrices of bench.py, device-resident
        _one("dev_1000sq_9pt", 9, (1000, 1000, 1)),
        _one("dev_64cube_27pt", 27, (64, 64, 64)),
        # many small matrices in one call: on the device, and a handful from host memory
        _many("batch512_dev", "batch", 512, 200, 5000, False),
        _many("batch10_host", "batch", 10, 200, 5000, True),
        # a burst of requests of the served mix, 10^3 to 10^5 rows
        _many("serve10", "serve", 10, 1000, 100000, True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(["symbolic", "symbolic", "symbolic", "symbolic", "noalloc", "batch", "serve"])
    host = rng.random() < 0.4
    if mode == "batch":
        return _many(None, mode, _log_uniform(rng, 2, 10 if host else 400), 200, 5000, host)
    if mode == "serve":
        lo = _log_uniform(rng, 1000, 4000)
        return _many(None, mode, rng.randint(2, 10), lo, _log_uniform(rng, 2 * lo, 100000), True)
    kind = rng.choice([5, 9, 7, 27])
    nd = rng.random() < 0.85
    if mode == "noalloc":
        n = _log_uniform(rng, 1000, 20000 if kind in (5, 9) else 8000)
        host = False
    elif kind in (5, 9):
        n = _log_uniform(rng, 1000, 900000)
    else:
        n = _log_uniform(rng, 1000, 200000)
    if not nd:
        n = min(n, 4000)  # a natural ordering fills in by the grid's whole width
    if kind in (5, 9):
        nx = max(2, int(round(math.sqrt(n) * math.exp(rng.uniform(-0.4, 0.4)))))
        dims = (nx, max(2, n // nx), 1)
    else:
        nx = max(2, int(round(n ** (1 / 3) * math.exp(rng.uniform(-0.2, 0.2)))))
        ny = max(2, int(round(math.sqrt(n / nx) * math.exp(rng.uniform(-0.2, 0.2)))))
        dims = (nx, ny, max(2, n // (nx * ny)))
    return _one(None, kind, dims, nd=nd, host=host, l_csr=mode == "symbolic" and rng.random() < 0.25,
                supernodes=rng.random() < 0.8, max_supernode=rng.choice([0, 0, 16, 256]), mode=mode)


# ---- sizes of the matrices of a case (seed-independent)

def _member_grid(i, lo, hi):
    """Grid of the i-th small matrix of a batch: even 2D 5-point, odd 3D 7-point."""
    n = lo + synth.sm64(0x5EED + i) % (hi - lo + 1)
    return (5, synth.grid_2d(n) + (1,)) if i % 2 == 0 else (7, synth.grid_3d(n))


def _request_grid(i, count, lo, hi):
    """Grid of the i-th served request: sizes spread evenly over the logarithm,
    2D 9-point and 3D 27-point in turn, large and small ones interleaved."""
    k = (i * 7) % count if count % 7 else i
    n = int(round(lo * (hi / lo) ** (k / max(count - 1, 1))))
    return (9, synth.grid_2d(n) + (1,)) if i % 2 == 0 else (27, synth.grid_3d(n))


def _grids(case):
    if case["mode"] == "batch":
        return [_member_grid(i, case["n_lo"], case["n_hi"]) for i in range(case["count"])]
    if case["mode"] == "serve":
        return [_request_grid(i, case["count"], case["n_lo"], case["n_hi"]) for i in range(case["count"])]
    return [(case["kind"], (case["nx"], case["ny"], case["nz"]))]


@functools.lru_cache(maxsize=2048)
def _base(kind, dims, nd, index, extras):
    s = synth.sm64((0xCA5E << 32) + index)
    m = synth.stencil(kind, dims, nd=nd, seed=s)
    return synth.band_extras(m, (m.nnz - m.n) // 10, seed=s, bw=32) if extras else m


def _lone_rows(n):
    return 8 + n // 1000


def _with_lone_rows(m, rng):
    """m with _lone_rows(m.n) rows that hold a diagonal entry only, at random places."""
    pos = np.sort(rng.integers(0, m.n + 1, _lone_rows(m.n)))
    lone = pos + np.arange(len(pos))
    ids = np.arange(m.n) + np.searchsorted(pos, np.arange(m.n), side="right")
    n = m.n + len(pos)
    deg = np.ones(n, dtype=np.int64)
    deg[ids] = np.diff(m.row_ptr)
    row_ptr = np.zeros(n + 1, dtype=np.int32)
    row_ptr[1:] = np.cumsum(deg)
    col = np.insert(ids[m.col_idx], m.row_ptr[pos], lone).astype(np.int32)
    return synth.Matrix(n, row_ptr, col, m.desc)


def _matrices(case, seed):
    rng = np.random.default_rng(int(seed))
    extras = case["mode"] == "batch"
    return [_with_lone_rows(_base(kind, dims, case.get("nd", True), i, extras), rng)
            for i, (kind, dims) in enumerate(_grids(case))]


def _flags(case):
    f = 0
    if not case.get("host"):
        f |= g.RESULT_ON_DEVICE
    if case.get("l_csr"):
        f |= g.L_CSR
    if case.get("supernodes") is False:
        f |= g.NO_SUPERNODES
    return f


def _dev(m):
    return m.n, torch.from_numpy(m.row_ptr).cuda(), torch.from_numpy(m.col_idx).cuda()


def prepare(case, seed):
    mats = _matrices(case, seed)
    st = {"mode": case["mode"], "host": bool(case.get("host")), "flags": _flags(case),
          "stream": torch.cuda.current_stream().cuda_stream}
    # the number of supernodes depends on where rows lie: the partition goes to an
    # array of its largest size
    rows = sum(m.n for m in mats)
    if st["flags"] & g.NO_SUPERNODES:
        st["xsup"] = None
    elif st["host"]:
        st["xsup"] = [np.full(m.n + 1, -1, dtype=np.int32) for m in mats]
    else:
        st["xsup"] = torch.full((rows + len(mats),), -1, dtype=torch.int32, device="cuda")
    if case["mode"] == "serve":
        st["mats"] = [(m.n, m.row_ptr, m.col_idx) for m in mats]
        srv = g.Server(max_inflight=4)
        st["srv"] = srv
        st["close"] = weakref.finalize(srv, g.Server.close, _Handle(srv))
        return st
    st["mats"] = [(m.n, m.row_ptr, m.col_idx) if st["host"] else _dev(m) for m in mats]
    st["max_supernode"] = case.get("max_supernode", 0)
    if case["mode"] == "noalloc":
        n, rp, ci = st["mats"][0]
        st["flags"] &= ~g.RESULT_ON_DEVICE
        # a program learns the capacities from an earlier factorisation
        r = g.symbolic(n, rp, ci, flags=g.RESULT_ON_DEVICE | g.NO_TUNE, stream=st["stream"])
        caps = {"u_idx": r.nnz_u, "l_idx": max(r.nnz_l, 1)}
        r.free()
        out = {"u_ptr": torch.empty(n + 1, dtype=torch.int64, device="cuda"),
               "l_ptr": torch.empty(n + 1, dtype=torch.int64, device="cuda"),
               "u_idx": torch.empty(caps["u_idx"], dtype=torch.int32, device="cuda"),
               "l_idx": torch.empty(caps["l_idx"], dtype=torch.int32, device="cuda")}
        if not st["flags"] & g.NO_SUPERNODES:
            out["xsup"] = st["xsup"]
            out["supno"] = torch.empty(n, dtype=torch.int32, device="cuda")
        st["out"] = out
    return st


class _Handle:
    """What closing a server needs, without keeping the server object alive."""

    def __init__(self, srv):
        self._lib, self._h = srv._lib, srv._h


class _View:
    """A device array of a result, kept alive with it."""

    def __init__(self, hold, ptr, count, typestr):
        self._hold = hold
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": typestr, "data": (ptr, False), "version": 2}


def _tensor(hold, ptr, count, wide=False):
    if count <= 0 or not ptr:
        return torch.empty(0, dtype=torch.int64 if wide else torch.int32, device="cuda")
    return torch.as_tensor(_View(hold, ptr, count, "<i8" if wide else "<i4"), device="cuda")


def _views(hold, p, n_ptr, nnz_l, nnz_u, rows, n_xsup, xsup):
    out = {"l_ptr": _tensor(hold, p["l_ptr"], n_ptr, True), "u_ptr": _tensor(hold, p["u_ptr"], n_ptr, True),
           "l_idx": _tensor(hold, p["l_idx"], nnz_l), "u_idx": _tensor(hold, p["u_idx"], nnz_u)}
    if xsup is not None:
        xsup[:n_xsup].copy_(_tensor(hold, p["xsup"], n_xsup))
        out["xsup"], out["supno"] = xsup, _tensor(hold, p["supno"], rows)
    return out


def _host(r, xsup):
    out = {"l_ptr": r.l_ptr, "l_idx": r.l_idx, "u_ptr": r.u_ptr, "u_idx": r.u_idx}
    if xsup is not None:
        xsup[:r.nsuper + 1] = r.xsup
        out["xsup"], out["supno"] = xsup, r.supno
    return out


def _counts(rs):
    return np.array([[r.nnz_l, r.nnz_u, r.fills, r.nsuper, r.stats["edges_alg"]] for r in rs], dtype=np.int64)


def run(state):
    mode, flags, stream = state["mode"], state["flags"], state["stream"]
    mats, xsup = state["mats"], state["xsup"]
    if mode == "serve":
        srv = state["srv"]
        tickets = [srv.submit(*m) for m in mats]
        rs = [srv.poll(t, timeout_us=-1) for t in tickets]
        return {"results": [_host(r, x) for r, x in zip(rs, xsup)], "counts": _counts(rs)}
    if mode == "noalloc":
        n, rp, ci = mats[0]
        out = state["out"]
        c = g.symbolic_noalloc(n, rp, ci, **out, flags=flags, max_supernode=state["max_supernode"], stream=stream)
        got = dict(out)
        got["counts"] = np.array([c["nnz_l"], c["nnz_u"], c["fills"], c["nsuper"], c["stats"]["edges_alg"]])
        return got
    if mode == "batch":
        rs = g.batch(mats, flags=flags, stream=stream)
        if state["host"]:
            return {"results": [_host(r, x) for r, x in zip(rs, xsup)], "counts": _counts(rs)}
        # the matrices' arrays lie side by side, in the order of the batch
        counts = _counts(rs)
        rows, nnz = sum(m[0] for m in mats), counts.sum(axis=0)
        first, last = rs[0].ptrs, rs[-1].ptrs
        for k, total, own in (("l_idx", nnz[0], counts[-1][0]), ("u_idx", nnz[1], counts[-1][1])):
            if last[k] - first[k] != 4 * (int(total) - int(own)):
                raise RuntimeError(f"{k} of the batch is not contiguous")
        out = _views(rs, first, rows + len(mats), int(nnz[0]), int(nnz[1]), rows, int(nnz[3]) + len(mats), xsup)
        out["counts"] = counts
        return out
    n, rp, ci = mats[0]
    r = g.symbolic(n, rp, ci, flags=flags, max_supernode=state["max_supernode"], stream=stream)
    if state["host"]:
        return dict(_host(r, xsup[0] if xsup else None), counts=_counts([r]))
    out = _views(r, r.ptrs, n + 1, r.nnz_l, r.nnz_u, n, r.nsuper + 1, xsup)
    out["counts"] = _counts([r])
    return out


# ---- work of a pass

POINTS = {5: 4, 9: 8, 7: 6, 27: 26}


def _entries(kind, dims, nd, extras):
    """(stored entries, entries of L and U): the stored ones from the grid, the
    factors' from fits of the generated stencils (within about 5 %; natural
    orderings and batch members within about 15 %)."""
    nx, ny, nz = dims
    n = nx * ny * nz
    nnz = 1 + 0.8 * POINTS[kind] * (0.9 if extras else 1.0) + (0.1 * 0.8 * POINTS[kind] if extras else 0.0)
    if not nd:
        band = sorted(dims)[-2] * (1 if nz == 1 else sorted(dims)[0])
        per = min(1.45 * band, n)
    elif nz == 1:
        per = (6.9 * math.log2(n) - 36 if kind == 9 else 5.2 * math.log2(n) - 29.6) if n > 200 else 10
    else:
        a = n ** (1 / 3)
        per = a * max(21.5 - 95 / a if kind == 27 else 15.3 - 78 / a, 3.0)
    return n * nnz, n * per * (2.7 if extras else 1.0)


def work(case):
    """Bytes of one pass: each matrix's CSR read once, its L and U indices,
    pointers and supernode partition written once. Index work only, no
    floating-point operations."""
    b = 0.0
    for kind, dims in _grids(case):
        n = dims[0] * dims[1] * dims[2]
        nnz, filled = _entries(kind, dims, case.get("nd", True), case["mode"] == "batch")
        n, nnz, filled = (v + _lone_rows(n) for v in (n, nnz, filled))
        b += 4 * (n + 1 + nnz) + 16 * (n + 1) + 4 * filled
        if case.get("supernodes", True):
            b += 6 * n
    return {"bytes": b, "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number: nothing is rounded."""
    return None
