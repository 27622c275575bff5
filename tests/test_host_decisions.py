"""Decisions of the library compiled for the host from the header that its own
code uses. The device's input check reads a row's columns only if a predicate
admits it: whatever row_ptr holds, no admitted row leaves the entries, and of a
non-decreasing row_ptr every row is admitted. After a launch of the block path:
a wait that gave up or a pool that cannot grow leaves the call to the traversal."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_00840_amd", "csrc")


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    d = tmp_path_factory.mktemp("checks")
    src, lib = d / "checks.cpp", d / "checks.so"
    src.write_text('#include "gsofa_checks.h"\n'
                   'extern "C" int row(int64_t r, int32_t a, int32_t b, int32_t nnz)\n'
                   '{ return gsofa::csr_row_readable(r, a, b, nnz); }\n'
                   'extern "C" int next(int how, int fits)\n'
                   '{ const uint32_t code[] = {gsofa::kBmNoAbort, gsofa::kBmOverflow, gsofa::kBmStall};\n'
                   '  return (int)gsofa::bm_next(code[how], fits != 0); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


@pytest.fixture(scope="module")
def readable(checks):
    fn = checks.row
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


def test_what_follows_a_launch(checks):
    results, again, traverse = range(3)
    done, overflow, stall = range(3)
    assert [checks.next(done, f) for f in (0, 1)] == [results, results]
    assert [checks.next(overflow, f) for f in (0, 1)] == [traverse, again]
    assert [checks.next(stall, f) for f in (0, 1)] == [traverse, traverse]


def test_bench_reads_the_block_path_s_traffic_record():
    """bench.py reports the committed counters of k_bm_factor only for the workload and
    the workgroups they were taken with, and while the kernel source is the same."""
    import re
    import sys
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench
    text = open(os.path.join(ROOT, "profiles", "k_bm_blocks.md")).read()
    recs = re.findall(r"traffic-record: workload=(\S+) kernel=(\S+) source_sha256_16=(\S+) sources=(\d+) "
                      r"fetch_bytes=(\d+) write_bytes=(\d+)", text)
    assert {r[0] for r in recs} == {"3d", "2d"}
    for workload, kernel, sha, sources, fetch, write in recs:
        got = bench.recorded_traffic(kernel, bench.MAP_BLOCKS, 0, int(sources), workload)
        assert got == (int(fetch) + int(write) if sha == bench.block_source_hash() else None)
        assert bench.recorded_traffic(kernel, bench.MAP_BLOCKS, 0, int(sources) + 64, workload) is None
