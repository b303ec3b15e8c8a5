"""The search by which a wavefront finds its rows, run on the host: every lane of every round looks inside the row pointers, and the place is
the first one that reaches the target.  Both ends of a chunk are searched together, so the one that is found first is asked again."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_15155_amd", "csrc")
HARNESS = """
#define __host__
#define __device__
#include "row_search.h"
using sensei::RowSearch;
// places found by the two searches; the number of looks outside [0, n] (not read)
extern "C" long search(const int *row_ptr, int n, long t0, long t1, int *found) {
    RowSearch s[2] = {{0, n}, {0, n}};
    const long t[2] = {t0, t1};
    long outside = 0;
    while (s[0].open() || s[1].open())
        for (auto &x : s) {
            int smaller = 0;
            for (int lane = 0; lane < 64; ++lane) {
                const int p = x.place(lane);
                if (p < 0 || p > n) { ++outside; continue; }
                smaller += p < x.hi && row_ptr[p] < t[&x - s];
            }
            x.narrow(smaller);
        }
    found[0] = s[0].lo;
    found[1] = s[1].lo;
    return outside;
}
"""


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_search")
    src, so = str(d / "harness.cpp"), str(d / "harness.so")
    with open(src, "w") as f:
        f.write(HARNESS)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-I" + CSRC, src, "-o", so])
    fn = C.CDLL(so).search
    fn.restype, fn.argtypes = C.c_long, [C.c_void_p, C.c_int, C.c_long, C.c_long, C.c_void_p]
    return fn


# 65 rows: the first end is found in one round and the second takes another
@pytest.mark.parametrize("n", [0, 1, 2, 63, 64, 65, 66, 129, 130, 131, 4_224, 4_225, 4_226, 8_450, 100_000, 274_625])
@pytest.mark.parametrize("mean", [0, 0.4, 1, 7])
@pytest.mark.parametrize("hub", [False, True])
def test_looks_stay_inside_and_find_the_row(search, n, mean, hub):
    rng = np.random.default_rng(n)
    deg = rng.poisson(mean, n)
    deg[: n // 5] = 0   # empty rows at the start
    if hub and n > 2:
        deg[n // 2] += 1_000
    row_ptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    found, nnz = np.empty(2, np.int32), int(row_ptr[-1])
    for t0 in sorted({0, 64, nnz // 2 // 64 * 64, nnz // 64 * 64}):
        assert search(row_ptr.ctypes.data, n, t0, t0 + 64, found.ctypes.data) == 0
        expected = np.searchsorted(row_ptr, [t0, t0 + 64], side="left")   # first place that reaches the target
        assert list(found) == list(np.minimum(expected, n))
