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
