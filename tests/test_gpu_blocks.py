"""The block path (64 rows at a time as bit masks) at the sizes where it can go
wrong: edges of blocks and tiles, lists of more than 64 tiles, column ranges of
more than 1,024 tiles, patterns without symmetry, pool regrowth. Every array and
edges_alg equal the oracle's exactly (whole numbers), and the per-source
traversal's."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2007_00840_amd as g
    g.load()
    return g


def _csr(n, rows):
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum([len(r) for r in rows])
    return n, rp, np.concatenate([np.asarray(r, dtype=np.int32) for r in rows]).astype(np.int32)


def _stencil(kind, dims, nd, seed):
    m = synth.stencil(kind, dims, nd=nd, seed=seed)
    return m.n, m.row_ptr, m.col_idx


def _band(n, below, above, seed):
    """Random band without symmetry, shuffled columns, some rows without diagonal."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(n):
        c = np.arange(max(0, i - below), min(n, i + above + 1))
        c = c[rng.random(len(c)) < 0.4]
        rows.append(rng.permutation(c))
    return _csr(n, rows)


def _random(n, per_row, seed):
    rng = np.random.default_rng(seed)
    return _csr(n, [rng.choice(n, per_row, replace=False) for _ in range(n)])


def _last_row_dense(n):
    """One row block with entries in every column tile before it."""
    rows = [[i] for i in range(n - 1)] + [list(range(n))]
    return _csr(n, rows)


def _first_column_dense(n):
    """One column with entries in every row block."""
    return _csr(n, [[0]] + [[0, i] for i in range(1, n)])


def _dense_rows(n, every):
    """Every `every`-th row holds all columns before it: many L tiles per block
    and no fill."""
    return _csr(n, [list(range(i + 1)) if i % every == every - 1 else [i] for i in range(n)])


CASES = {
    **{f"band_n{n}": lambda n=n: _band(n, 9, 11, n) for n in (1, 2, 63, 64, 65, 127, 128, 129, 200)},
    "band_lower": lambda: _band(700, 40, 0, 1),
    "band_upper": lambda: _band(700, 0, 40, 2),
    "band_wide": lambda: _band(1500, 150, 90, 3),
    "random_filled": lambda: _random(900, 4, 4),
    "nd_2d": lambda: _stencil(9, (70, 61), True, 5),
    "nd_3d": lambda: _stencil(27, (19, 18, 17), True, 6),
    "natural_3d": lambda: _stencil(7, (13, 12, 11), False, 7),
    "last_row_dense": lambda: _last_row_dense(70000),
    "first_column_dense": lambda: _first_column_dense(70000),
    "pool_regrowth": lambda: _dense_rows(24576, 64),
    "pairs": lambda: _pairs(20000, 9),
}


@pytest.mark.parametrize("name", CASES)
def test_block_path_matches_oracle(g, name):
    n, rp, ci = CASES[name]()
    print(f"blocks {name} n={n} nnz={len(ci)}", flush=True)
    sys.stdout.flush()
    ref = oracle.symbolic(n, rp, ci)
    fills = oracle.fills(ref, rp, ci)
    for flags in (0, g.L_CSR):
        r = g.symbolic(n, rp, ci, flags=flags)
        assert r.stats["mapping"] == 7
        assert np.array_equal(r.u_ptr, ref.u_ptr) and np.array_equal(r.u_idx, ref.u_idx)
        assert np.array_equal(r.l_ptr, ref.l_rptr if flags else ref.l_ptr)
        assert np.array_equal(r.l_idx, ref.l_ridx if flags else ref.l_idx)
        assert np.array_equal(r.xsup, ref.xsup) and np.array_equal(r.supno, ref.supno)
        assert r.stats["edges_alg"] == ref.edges_alg and r.fills == fills
    t = g.symbolic(n, rp, ci, flags=g.MAP_WAVE32)
    assert t.stats["mapping"] == 0
    assert np.array_equal(t.u_idx, ref.u_idx) and t.fills == fills


def test_block_path_repeated_column_is_refused(g):
    n, rp, ci = _stencil(9, (20, 20), True, 8)
    ci = ci.copy()
    ci[rp[7] + 1] = ci[rp[7]]
    import torch
    with pytest.raises(g.GsofaError) as e:
        g.symbolic(n, torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda())
    assert e.value.code == g.EINVAL
    n, rp, ci = _stencil(9, (20, 20), True, 8)
    assert g.symbolic(n, rp, ci).fills == oracle.fills(oracle.symbolic(n, rp, ci), rp, ci)


def _pairs(n, seed):
    """Rows coupled two by two at random: a tile per entry, which the block path's
    share of the fixed scratch does not hold."""
    p = np.random.default_rng(seed).permutation(n)
    mate = np.empty(n, dtype=np.int64)
    mate[p[0::2]], mate[p[1::2]] = p[1::2], p[0::2]
    rows = np.sort(np.stack([np.arange(n), mate], axis=1), axis=1)
    return n, np.arange(0, 2 * n + 1, 2, dtype=np.int32), rows.reshape(-1).astype(np.int32)


NOALLOC = {
    **{f"band_n{n}": (lambda n=n: _band(n, 9, 11, n), {}, 7) for n in (1, 63, 64, 65, 129)},
    "nd_2d": (lambda: _stencil(9, (70, 61), True, 5), {}, 7),
    "nd_3d": (lambda: _stencil(27, (19, 18, 17), True, 6), {}, 7),
    "sources_named": (lambda: _stencil(9, (70, 61), True, 5), {"concurrent_sources": 64}, 0),
    "window_named": (lambda: _stencil(9, (70, 61), True, 5), {"window": 16}, 0),
    "tiles_do_not_fit": (lambda: _pairs(200000, 9), {}, 0),
}


@pytest.mark.parametrize("name", NOALLOC)
def test_noalloc_path_and_result(g, name):
    import torch
    make, opts, mapping = NOALLOC[name]
    n, rp, ci = make()
    print(f"noalloc {name} n={n} nnz={len(ci)}", flush=True)
    ref = oracle.symbolic(n, rp, ci)
    # (one entry more than the matrix has: an empty tensor has no address)
    drp, dci = torch.from_numpy(rp).cuda(), torch.from_numpy(np.append(ci, np.int32(0))).cuda()
    nu, nl = int(ref.u_ptr[-1]), int(ref.l_ptr[-1])
    for flags in (0, g.L_CSR):
        out = {k: torch.full((m,), -7, dtype=t, device="cuda")
               for k, m, t in (("u_ptr", n + 1, torch.int64), ("l_ptr", n + 1, torch.int64),
                               ("u_idx", nu + 3, torch.int32), ("l_idx", nl + 3, torch.int32),
                               ("xsup", n + 1, torch.int32), ("supno", n, torch.int32))}
        c = g.symbolic_noalloc(n, drp, dci, **out, flags=flags, **opts)
        assert c["stats"]["mapping"] == mapping
        got = {k: v.cpu().numpy() for k, v in out.items()}
        assert (c["nnz_u"], c["nnz_l"], c["stats"]["edges_alg"]) == (nu, nl, ref.edges_alg)
        assert np.array_equal(got["u_ptr"], ref.u_ptr) and np.array_equal(got["u_idx"][:nu], ref.u_idx)
        assert np.array_equal(got["l_ptr"], ref.l_rptr if flags else ref.l_ptr)
        assert np.array_equal(got["l_idx"][:nl], ref.l_ridx if flags else ref.l_idx)
        assert np.array_equal(got["xsup"][:c["nsuper"] + 1], ref.xsup) and np.array_equal(got["supno"], ref.supno)
        assert (got["u_idx"][nu:] == -7).all() and (got["l_idx"][nl:] == -7).all()
    # the limits are those of the traversal: what it refuses for want of room is
    # refused here with the same totals
    small = dict(out, u_idx=out["u_idx"][:max(nu - 1, 0)])
    counts = []
    for o in (opts, dict(opts, concurrent_sources=1 << 20)):
        with pytest.raises(g.GsofaError) as e:
            g.symbolic_noalloc(n, drp, dci, **small, **o)
        assert e.value.code == g.ECAPACITY
        counts.append([e.value.counts[k] for k in ("nnz_u", "nnz_l", "fills", "scratch_bytes")])
    if "concurrent_sources" not in opts:
        assert counts[0] == counts[1]


SUPERNODES = {
    "dense": lambda: _csr(300, [list(range(300)) for _ in range(300)]),
    "band_lower": lambda: _band(700, 40, 0, 1),
    "band_wide": lambda: _band(1500, 150, 90, 3),
    "nd_3d": lambda: _stencil(27, (19, 18, 17), True, 6),
    "n64": lambda: _band(64, 9, 11, 64),
    "n65": lambda: _band(65, 30, 30, 65),
}


@pytest.mark.parametrize("name", SUPERNODES)
def test_block_supernodes_match_traversal(g, name):
    """Chains that cross blocks of rows, at limits below, at and above a block."""
    n, rp, ci = SUPERNODES[name]()
    print(f"supernodes {name} n={n}", flush=True)
    for limit in (1, 50, 64, 65, 200, -1):
        for flags in (0, g.L_CSR):
            r = g.symbolic(n, rp, ci, flags=flags, max_supernode=limit)
            t = g.symbolic(n, rp, ci, flags=flags | g.MAP_WAVE32, max_supernode=limit)
            assert (r.stats["mapping"], t.stats["mapping"]) == (7, 0)
            assert np.array_equal(r.xsup, t.xsup) and np.array_equal(r.supno, t.supno), limit


@pytest.mark.parametrize("n", [8191, 8192, 8193, 3 * 8192 + 5])
def test_block_sums_at_tile_edges(g, n):
    """Row counts, columns and supernode starts are summed in tiles of 8,192; a
    batch also by its blocks and between its matrices."""
    rp, ci = np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32)
    small = _band(129, 9, 11, n)
    r = g.symbolic(n, rp, ci)
    assert r.stats["mapping"] == 7 and r.nsuper == n
    assert np.array_equal(r.u_ptr, np.arange(n + 1)) and np.array_equal(r.u_idx, ci) and r.nnz_l == 0
    assert np.array_equal(r.supno, ci) and np.array_equal(r.xsup, np.arange(n + 1))
    ref = oracle.symbolic(*small)
    for a, b in zip(g.batch([small, (n, rp, ci), small]), (ref, r, ref)):
        assert np.array_equal(a.u_ptr, b.u_ptr) and np.array_equal(a.l_ptr, b.l_ptr)
        assert np.array_equal(a.u_idx, b.u_idx) and np.array_equal(a.l_idx, b.l_idx)
        assert np.array_equal(a.xsup, b.xsup) and np.array_equal(a.supno, b.supno)


def test_malformed_device_input_is_told_apart(g):
    """A negative entry count is found without looking at anything else, and is
    then the only matrix of the batch that is refused."""
    import torch
    n, rp, ci = _stencil(9, (20, 20), True, 8)
    dev = lambda a: torch.from_numpy(a).cuda()
    good = (n, dev(rp), dev(ci))
    neg = rp.copy()
    neg[n] = -1
    off = ci.copy()
    off[3] = n
    for bad in ((n, dev(neg), dev(ci)), (n, dev(rp), dev(off))):
        with pytest.raises(g.GsofaError) as e:
            g.symbolic(*bad)
        assert e.value.code == g.EINVAL
        r = g.batch([good, bad, good], raise_on_error=False)
        assert r[1] is None
    both = g.batch([(n, dev(rp), dev(off)), (n, dev(neg), dev(ci))], raise_on_error=False)
    assert both[1] is None
    assert g.symbolic(*good).fills == g.symbolic(n, rp, ci).fills


def test_row_pointers_beyond_the_entries_are_refused(g):
    """A row that ascends on its own but ends beyond row_ptr[n]: refused without a
    read of the columns there (the bound itself is tested on the host), by every
    entry point that takes device arrays."""
    import torch
    n, rp, ci = _stencil(9, (20, 20), True, 8)
    dev = lambda a: torch.from_numpy(a).cuda()
    for at in (1, n // 2, n - 1):
        far = rp.copy()
        far[at] = 1 << 30
        bad = (n, dev(far), dev(ci))
        with pytest.raises(g.GsofaError) as e:
            g.symbolic(*bad)
        assert e.value.code == g.EINVAL
        assert g.batch([bad], raise_on_error=False) == [None]
        out = {k: torch.zeros(m, dtype=t, device="cuda")
               for k, m, t in (("u_ptr", n + 1, torch.int64), ("l_ptr", n + 1, torch.int64),
                               ("u_idx", 4, torch.int32), ("l_idx", 4, torch.int32),
                               ("xsup", n + 1, torch.int32), ("supno", n, torch.int32))}
        with pytest.raises(g.GsofaError) as e:
            g.symbolic_noalloc(*bad, **out)
        assert e.value.code == g.EINVAL


@pytest.mark.parametrize("path", ["blocks", "traversal"])
def test_largest_order_and_entry_count(g, path):
    """2^22 rows, the most the block path takes, in dense blocks of 512 with
    2^31 - 1 entries in all: the last step over a row's (block's) entries passes 2^31."""
    import torch
    n, nnz = 1 << 22, 2**31 - 1
    ci = torch.empty(nnz, dtype=torch.int32, device="cuda")
    step = 1 << 28
    for a in range(0, nnz, step):
        i = torch.arange(a, min(a + step, nnz), device="cuda")
        ci[a:a + step] = ((i >> 18 << 9) + (i & 511)).to(torch.int32)
    r = torch.arange(n + 1, device="cuda")
    rp = (512 * r).clamp(max=nnz).to(torch.int32)
    print(f"{path} n={n} nnz={nnz}", flush=True)
    flags, mapping = {"blocks": (0, 7), "traversal": (g.MAP_WAVE32, 0)}[path]
    d = g.symbolic(n, rp, ci, flags=g.RESULT_ON_DEVICE | flags)
    assert d.stats["mapping"] == mapping and d.fills == 0
    assert (d.nnz_u, d.nnz_l, d.nsuper) == (n // 512 * (512 * 513 // 2), n // 512 * (512 * 511 // 2), n // 128)
    # every source reaches the rows of its dense block above it, 512 entries each
    # (the last row, only a source, lacks one)
    assert d.stats["edges_alg"] == n // 512 * 512 * (512 * 513 // 2) - 1
    t = d.to_torch()
    d.free()
    m = torch.arange(512, device="cuda")
    at = torch.cat([m.new_zeros(1), (512 - m).cumsum(0)])  # of a block's rows of U
    assert torch.equal(t["u_ptr"], (r >> 9) * at[512] + at[r & 511])
    at = torch.cat([m.new_zeros(1), (511 - m).cumsum(0)])  # of its columns of L
    assert torch.equal(t["l_ptr"], (r >> 9) * at[512] + at[r & 511])
    for k, first in (("u_idx", 0), ("l_idx", 1)):
        one = torch.cat([m[c + first:] for c in range(512)])
        x = t[k].view(n // 512, -1)
        for a in range(0, n // 512, 1024):
            want = one[None] + 512 * torch.arange(a, a + 1024, device="cuda")[:, None]
            assert torch.equal(x[a:a + 1024], want.to(torch.int32)), (k, a)
    del t, ci
    g.release_cache()


@pytest.mark.parametrize("nd", [1, 2])
def test_batch_with_a_member_of_more_than_2_21_rows(g, nd):
    """The bitmaps of 2^21 rows and more leave room for four wavefronts per block."""
    n = (1 << 21) + 64 * nd + 5
    big = (n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32)[::-1].copy())
    small = _band(129, 9, 11, nd)
    ref = oracle.symbolic(*small)
    a, b = g.batch([small, big])
    assert (a.stats["mapping"], b.stats["mapping"]) == (7, 7)
    assert np.array_equal(a.u_idx, ref.u_idx) and np.array_equal(a.l_idx, ref.l_idx)
    # row i holds column n - 1 - i: an entry of U above the middle, of L below it,
    # whose row n - 1 - i holds nothing beyond its own diagonal
    i = np.arange(n)
    assert np.array_equal(b.u_ptr, np.concatenate([[0], np.cumsum(np.where(i < n // 2, 2, 1))]))
    assert np.array_equal(b.l_ptr, np.concatenate([[0], np.cumsum(np.where(i < n // 2, 1, 0))]))
    assert np.array_equal(b.l_idx, n - 1 - i[:n // 2])
    assert b.fills == 0


def _same(r, ref):
    assert np.array_equal(r.u_ptr, ref.u_ptr) and np.array_equal(r.u_idx, ref.u_idx)
    assert np.array_equal(r.l_ptr, ref.l_ptr) and np.array_equal(r.l_idx, ref.l_idx)
    assert np.array_equal(r.xsup, ref.xsup) and np.array_equal(r.supno, ref.supno)
    assert r.stats["edges_alg"] == ref.edges_alg


def test_memory_that_cannot_be_had_leaves_the_call_to_the_traversal(g):
    """One request of a caller's allocator fails, at several places of the call."""
    m = _stencil(9, (70, 61), True, 5)
    ref = oracle.symbolic(*m)

    class Failing(g.TorchAllocator):
        def __init__(self, at):
            super().__init__()
            self.asked, inner = 0, self.alloc_fn

            def alloc(nbytes, ctx):
                self.asked += 1
                return None if self.asked == at else inner(nbytes, ctx)
            self._inner, self.alloc_fn = inner, g.ALLOC_FN(alloc)

    al = Failing(0)
    r = g.symbolic(*m, allocator=al)
    assert r.stats["mapping"] == 7
    _same(r, ref)
    inputs = 3  # row pointers, columns, the job table
    for at in (inputs + 1, al.asked // 2, al.asked - 2, al.asked):
        print(f"allocation {at} of {al.asked} fails", flush=True)
        f = Failing(at)
        r = g.symbolic(*m, allocator=f)
        assert r.stats["mapping"] != 7
        _same(r, ref)
        assert f.frees == f.allocs and not f.live


def test_little_device_memory_free(g):
    """A call whose planned workgroups do not fit the free memory runs with fewer."""
    import torch
    n, rp, ci = _stencil(9, (350, 350), True, 5)
    g.symbolic(n, rp, ci)  # (the first call of a size class takes more tiles)
    full = g.symbolic(n, rp, ci)
    assert full.stats["mapping"] == 7
    need = full.stats["peak_device_bytes"]
    g.release_cache()
    torch.cuda.empty_cache()
    free = lambda: torch.cuda.mem_get_info()[0]
    held = []
    try:
        while free() > need and len(held) < 8:
            held.append(torch.empty(free() - need + (1 << 22), dtype=torch.uint8, device="cuda"))
        print(f"free {free()} of {need} that a call takes", flush=True)
        r = g.symbolic(n, rp, ci)
    finally:
        del held
        torch.cuda.empty_cache()
    assert r.stats["mapping"] == 7 and r.stats["concurrent_sources"] < full.stats["concurrent_sources"]
    for k in ("u_ptr", "u_idx", "l_ptr", "l_idx", "xsup", "supno"):
        assert np.array_equal(getattr(r, k), getattr(full, k)), k


def test_the_budget_holds_the_result_too(g):
    """A call with a budget takes the block path only where what it holds at a time,
    its result included, is within the budget: refused before the launch where the
    size class tells, after it where the result turns out larger."""
    n, rp, ci = _random(12000, 5, 11)  # 60,000 entries fill to some 60 million
    full = g.symbolic(n, rp, ci, flags=g.NO_TUNE)
    out = 4 * (full.nnz_u + full.nnz_l)
    assert full.stats["mapping"] == 7 and full.stats["peak_device_bytes"] > out > 64 << 20
    few = _band(n, 6, 6, 3)  # of the same size class, with a small result
    paths = []
    for budget in (72 << 20, out, out + (64 << 20), 2 * out + (128 << 20)):
        for warm in ((n, rp, ci), few):  # what the class had last
            g.symbolic(*warm, flags=g.NO_TUNE)
            r = g.symbolic(n, rp, ci, flags=g.NO_TUNE, mem_budget_bytes=budget)
            paths.append(r.stats["mapping"])
            print(f"budget {budget >> 20} MiB of {out >> 20}: path {paths[-1]}", flush=True)
            assert r.stats["mapping"] != 7 or r.stats["peak_device_bytes"] <= budget
            for k in ("u_ptr", "u_idx", "l_ptr", "l_idx", "xsup", "supno"):
                assert np.array_equal(getattr(r, k), getattr(full, k)), k
            assert r.stats["edges_alg"] == full.stats["edges_alg"]
    assert paths[:4] == [0, 0, 0, 0] and paths[-2:] == [7, 7]
    # the masks of the launches that were given up are clean
    _same(g.symbolic(*few), oracle.symbolic(*few))


def test_a_served_request_larger_than_its_estimate(g):
    """The server runs it all the same, and has its whole budget back afterwards."""
    m, few = _random(12000, 5, 11), _band(12000, 6, 6, 3)
    ref = g.symbolic(*m)
    with g.Server(max_inflight=2, mem_budget_bytes=200 << 20) as s:
        for _ in range(4):
            g.symbolic(*few)  # (estimates follow the last result)
            r = s.poll(s.submit(*m), timeout_us=-1)
            assert r.stats["mapping"] == 7 and r.stats["peak_device_bytes"] > 200 << 20
            assert np.array_equal(r.u_idx, ref.u_idx)


def test_a_budgeted_call_does_not_tune_others_off_the_path(g):
    """A call whose budget does not hold the block path may time the tuner's trials;
    what they choose holds for traversals, later default calls of the size class
    take the block path."""
    m = _pairs(70000, 10)
    a = g.symbolic(*m, mem_budget_bytes=110 << 20)
    assert a.stats["mapping"] != 7 and a.stats["t_tune_ms"] > 0
    b = g.symbolic(*m)
    assert b.stats["mapping"] == 7
    c = g.symbolic(*m, mem_budget_bytes=110 << 20)
    assert c.stats["mapping"] == a.stats["mapping"] and c.stats["t_tune_ms"] == 0
    for r in (a, c):
        for k in ("u_ptr", "u_idx", "l_ptr", "l_idx", "xsup", "supno"):
            assert np.array_equal(getattr(r, k), getattr(b, k)), k


def test_pool_regrowth_is_paid_once_per_size_class(g):
    """A first call of a class whose blocks have 312 tiles on average (the first pool
    holds at most 156 a block) runs its launch again, the next one does not; a 2D
    matrix between two 3D ones of its class leaves the pool as it is."""
    n, rp, ci = _dense_rows(40000, 64)
    first = g.symbolic(n, rp, ci, flags=g.NO_TUNE)
    again = g.symbolic(n, rp, ci, flags=g.NO_TUNE)
    assert (first.stats["mapping"], again.stats["mapping"]) == (7, 7)
    assert first.stats["launches"] >= 2 and again.stats["launches"] == 1
    nnz_l = len(ci) - n  # (no fill)
    for r in (first, again):
        assert r.fills == 0 and r.nnz_l == nnz_l and np.array_equal(r.u_idx, np.arange(n))
    m3, m2 = _stencil(7, (64, 64, 64), True, 5), _stencil(9, (510, 510), True, 5)
    a = g.symbolic(*m3, flags=g.NO_TUNE)
    for _ in range(2):
        assert g.symbolic(*m2, flags=g.NO_TUNE).stats["mapping"] == 7
    b = g.symbolic(*m3, flags=g.NO_TUNE)
    assert b.stats["launches"] == 1 and np.array_equal(a.u_idx, b.u_idx) and np.array_equal(a.l_idx, b.l_idx)


def test_pool_regrowth_in_a_batch(g):
    """The launch of all members runs again, the small ones' results with it."""
    n, rp, ci = _dense_rows(30000, 64)
    small = [_band(k, 9, 11, k) for k in (64, 129, 700)]
    res = g.batch([small[0], (n, rp, ci), small[1], small[2]], flags=g.NO_TUNE)
    assert res[0].stats["mapping"] == 7 and res[0].stats["launches"] >= 2
    assert res[1].fills == 0 and np.array_equal(res[1].u_idx, np.arange(n))
    for m, r in zip(small, (res[0], res[2], res[3])):
        _same(r, oracle.symbolic(*m))


def test_served_blocks_yield(g):
    """A large request on the block path (a tridiagonal matrix: 9,375 blocks one after
    another) gives the device up for requests admitted meanwhile with
    GSOFA_SERVE_YIELD: its launch stops taking blocks and is run again from there.
    Without the flag one launch does it all; the results are the same."""
    import time
    n = 600000
    i = np.arange(n)
    c = i[:, None] + np.arange(-1, 2)[None]
    ok = (c >= 0) & (c < n)
    rp = np.concatenate([[0], ok.sum(1).cumsum()]).astype(np.int32)
    tri = (n, rp, c[ok].astype(np.int32))
    small = [_band(700, 9, 11, k) for k in range(8)]
    refs = [oracle.symbolic(*m) for m in small]
    launches = {}
    for flags in (g.SERVE_YIELD, 0):
        with g.Server(max_inflight=4, flags=flags) as s:
            t = s.submit(*tri)
            ts = []
            for m in small:
                time.sleep(0.006)
                ts.append(s.submit(*m))
            r = s.poll(t, timeout_us=-1)
            rs = [s.poll(x, timeout_us=-1) for x in ts]
        launches[flags] = r.stats["launches"]
        print(f"flags {flags:#x}: {launches[flags]} launches", flush=True)
        assert r.stats["mapping"] == 7 and r.fills == 0 and r.nnz_l == n - 1
        assert np.array_equal(r.u_idx, c[ok & (c >= i[:, None])]) and np.array_equal(r.l_idx, i[1:])
        for x, ref in zip(rs, refs):
            _same(x, ref)
    assert launches[g.SERVE_YIELD] >= 2 and launches[0] == 1


def test_pool_of_a_small_call_grows(g):
    """24,000 rows with a dense first row and column fill up: the first pool is small
    enough for the device's free memory not to be asked for, the next one is not."""
    import torch
    n = 24000
    first = np.arange(n)
    rest = np.stack([np.zeros(n - 1, dtype=np.int64), np.arange(1, n)], 1).reshape(-1)
    rp = np.concatenate([[0], n + 2 * np.arange(n)]).astype(np.int32)
    d = g.symbolic(n, torch.from_numpy(rp).cuda(), torch.from_numpy(np.concatenate([first, rest]).astype(np.int32)).cuda(),
                   flags=g.RESULT_ON_DEVICE)
    assert d.stats["mapping"] == 7 and d.stats["launches"] >= 2
    assert d.nnz_u == n * (n + 1) // 2 and d.nnz_l == n * (n - 1) // 2
    t = d.to_torch()
    d.free()
    k = torch.arange(n + 1, device="cuda")
    assert torch.equal(t["u_ptr"], k * n - k * (k - 1) // 2) and torch.equal(t["l_ptr"], k * (n - 1) - k * (k - 1) // 2)
    for r in (0, 1, 63, 64, 12345, n - 1):
        assert torch.equal(t["u_idx"][t["u_ptr"][r]:t["u_ptr"][r + 1]], k[r:n].int())
        assert torch.equal(t["l_idx"][t["l_ptr"][r]:t["l_ptr"][r + 1]], k[r + 1:n].int())


def _entries(n, cols):
    """A diagonal and the given columns per row (n x k, repeats dropped)."""
    c = np.sort(np.concatenate([np.arange(n)[:, None], cols], axis=1), axis=1)
    keep = np.ones_like(c, dtype=bool)
    keep[:, 1:] = c[:, 1:] != c[:, :-1]
    return n, np.concatenate([[0], keep.sum(1).cumsum()]).astype(np.int32), c[keep].astype(np.int32)


def _below(n, k, seed):
    return _entries(n, np.random.default_rng(seed).integers(0, np.maximum(np.arange(n), 1)[:, None], (n, k)))


def _tree(n, width, seed):
    """A symmetric tree, every parent at most `width` rows below its child."""
    p = np.minimum(n - 1, np.arange(n - 1) + 1 + np.random.default_rng(seed).integers(0, width, n - 1))
    rows = [[i] for i in range(n)]
    for i, j in enumerate(p):
        rows[i].append(j)
        rows[j].append(i)
    return _csr(n, [sorted(set(r)) for r in rows])


SPARSE = {
    "below_1": lambda: _below(12000, 1, 1),    # tiles of one entry, lists of more than 64
    "below_3": lambda: _below(3000, 3, 2),     # tiles of one and of several
    "anywhere": lambda: _entries(9000, np.random.default_rng(3).integers(0, 9000, (9000, 1))),
    "first_rows": lambda: _entries(9000, np.random.default_rng(4).integers(0, 40, (9000, 2))),
    "tree": lambda: _tree(9000, 1500, 5),
    "n65": lambda: _below(65, 1, 6),
}


@pytest.mark.parametrize("name", SPARSE)
def test_reach_counts_of_scattered_entries(g, name):
    m = SPARSE[name]()
    ref = oracle.symbolic(*m)
    small = _band(129, 9, 11, 1)
    print(f"scattered {name} n={m[0]} nnz={len(m[2])}", flush=True)
    for r in (g.symbolic(*m), g.batch([small, m, small])[1]):
        assert r.stats["mapping"] == 7
        _same(r, ref)


def test_malformed_members_of_a_device_batch_leave_the_others_alone(g):
    """Every malformed matrix is refused (out-of-range columns, a negative count, rows
    that end beyond the entries, a repeated column) and every other one computed."""
    import torch
    dev = lambda m: (m[0],) + tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in m[1:])
    n, rp, ci = _stencil(9, (20, 20), True, 8)
    off, neg, far, twice = ci.copy(), rp.copy(), rp.copy(), ci.copy()
    off[3], neg[n], far[5] = n, -1, 1 << 30
    twice[rp[7] + 1] = twice[rp[7]]
    bad = [(n, rp, off), (n, neg, ci), (n, far, ci), (n, rp, twice)]
    good = [_band(k, 9, 11, k) for k in (1, 64, 200, 700)]
    refs = [oracle.symbolic(*m) for m in good]
    for pick in ((0,), (1,), (2,), (3,), (0, 1), (0, 1, 2, 3)):
        mats = [x for k, m in enumerate(good) for x in ([m, bad[k]] if k in pick else [m])]
        for flags in (0, g.MAP_WAVE32):
            res = g.batch([dev(m) for m in mats], raise_on_error=False, flags=flags)
            assert [r is None for r in res] == [any(m is b for b in bad) for m in mats]
            for r, ref in zip([r for r in res if r is not None], refs):
                _same(r, ref)
    with pytest.raises(g.GsofaError) as e:
        g.batch([dev(good[0]), dev(bad[0])])
    assert e.value.code == g.EINVAL
