"""Places of the pad rows' bin offsets in the slot's table, at the limits of a
slot: the arithmetic of csrc/bin_table.h, compiled for the CPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROWS = 36 * 159

SRC = r"""
#include "bin_table.h"
extern "C" uint32_t pair_of(uint32_t first, uint32_t sr) { return tpc::bin_table_pair(first, sr); }
extern "C" int64_t entries(int64_t n, int64_t rows) { return tpc::bin_table_entries(n, rows); }
extern "C" int per_hit() { return tpc::kBinsPerHit; }
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    d = tmp_path_factory.mktemp("bin_table")
    (d / "t.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1712_09416_amd", "csrc"), "-o", str(d / "t.so"), str(d / "t.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(d / "t.so"))
    lib.pair_of.argtypes = [ctypes.c_uint32, ctypes.c_uint32]
    lib.pair_of.restype = ctypes.c_uint32
    lib.entries.argtypes = [ctypes.c_int64, ctypes.c_int64]
    lib.entries.restype = ctypes.c_int64
    return lib


# one event of few clusters; a batch; more than 2^30 clusters, where a row's
# first entry is past 2^31; the most clusters and events a slot takes
@pytest.mark.parametrize("events,clusters", [(1, 0), (1, 1), (3, 20_000), (64, 1 << 30), (4096, 3 << 29),
                                             (128, 0x7FFFFFFF), (4096, 0x7FFFFFFF)])
def test_rows_do_not_share_entries(table, events, clusters):
    rng = np.random.default_rng(events)
    rows = events * ROWS
    # rows of very different sizes, empty ones among them
    cut = np.sort(rng.integers(0, clusters + 1, 2000))
    first = np.concatenate([[0], cut, [clusters]]).astype(np.int64)
    sr = np.sort(rng.choice(rows, 2001, replace=False)).astype(np.int64)
    sr[0], sr[-1] = 0, rows - 1
    n = np.diff(first)                  # row sr[k] has n[k] hits, the rows between have none
    start = np.array([2 * table.pair_of(int(f), int(s)) for f, s in zip(first, sr)])
    end = start + table.per_hit() * np.maximum(n, 1) + 1
    size = table.entries(clusters, rows)
    assert start[0] >= 0 and end.max() <= size and np.all(end[:-1] <= start[1:])
    # the empty rows between two of them
    gap = np.flatnonzero(np.diff(sr) > 1)
    nxt = np.array([2 * table.pair_of(int(first[k + 1]), int(sr[k] + 1)) for k in gap])
    assert np.all(nxt >= end[gap]) and np.all(nxt + table.per_hit() + 1 <= start[gap + 1])
