"""The check of host-side CSR input: rows in ascending order are recognised
without a look at each entry's history, all others are stamped. Repeated and
out-of-range columns are refused wherever they stand; order alone is no fault."""
import numpy as np
import pytest

import paper_2007_00840_amd as g

ROWS = [[0, 2, 5], [1], [], [0, 1, 2, 3, 4, 5, 6], [4], [5, 6], [6]]


def _code(rows, n=7):
    """GSOFA_OK, GSOFA_EINVAL or, where there is no device, GSOFA_EDEVICE."""
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum([len(r) for r in rows])
    ci = np.concatenate([np.asarray(r, dtype=np.int32) for r in rows]).astype(np.int32)
    try:
        g.symbolic(n, rp, ci)
    except g.GsofaError as e:
        return e.code
    return g.OK


@pytest.mark.parametrize("row", [0, 1, 3, 5, 6])
def test_repeats_and_range(row):
    for change in (lambda r: r + [r[-1]], lambda r: [r[-1]] + r, lambda r: r + [7], lambda r: r + [-1],
                   lambda r: r[::-1] + [r[0]]):
        rows = [list(r) for r in ROWS]
        rows[row] = change(rows[row])
        assert _code(rows) == g.EINVAL, rows[row]


@pytest.mark.parametrize("rows", [ROWS, [r[::-1] for r in ROWS], [[5, 0, 2]] + ROWS[1:], ROWS[:6] + [[6, 0]]])
def test_order_is_free(rows):
    assert _code(rows) != g.EINVAL
