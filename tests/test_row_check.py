"""The predicate by which the device's input check decides whether a row's
columns may be read, compiled for the host (the kernel uses the same header):
whatever row_ptr holds, no admitted row leaves the entries, and of a
non-decreasing row_ptr every row is admitted."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_00840_amd", "csrc")


@pytest.fixture(scope="module")
def readable(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    src, lib = d / "rows.cpp", d / "rows.so"
    src.write_text('#include "gsofa_checks.h"\n'
                   'extern "C" int row(int64_t r, int32_t a, int32_t b, int32_t nnz)\n'
                   '{ return gsofa::csr_row_readable(r, a, b, nnz); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(lib)], check=True)
    fn = ctypes.CDLL(str(lib)).row
    fn.argtypes = [ctypes.c_int64] + 3 * [ctypes.c_int32]
    return lambda rp: [bool(fn(r, int(rp[r]), int(rp[r + 1]), int(rp[-1]))) for r in range(len(rp) - 1)]


@pytest.mark.parametrize("rp", [[0, 1 << 30, 5], [0, 3, 2**31 - 1, 4], [0, 6, 5], [7, 9, 3], [-4, 2, 2],
                                [0, 2, -1, 4], [0, 2**31 - 1, -2**31, 1]])
def test_no_admitted_row_leaves_the_entries(readable, rp):
    rows = readable(rp)
    assert not all(rows)  # and the matrix is refused
    for r, ok in enumerate(rows):
        assert not ok or (0 <= rp[r] <= rp[r + 1] <= rp[-1])


def test_rows_of_random_pointers(readable):
    rng = np.random.default_rng(1)
    for _ in range(200):
        rp = rng.integers(-3, 12, 6)
        rows = readable(rp)
        for r, ok in enumerate(rows):
            assert not ok or (0 <= rp[r] <= rp[r + 1] <= rp[-1])
        up = np.sort(np.abs(rp)) - np.abs(rp).min()
        assert all(readable(up))
