"""Ranks that are used as places: for any values they are a permutation, NaN
last, ties by index (the header alone, compiled for the host)."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1004_3980_amd", "csrc")
SRC = """
#include "zh_order.h"
extern "C" void ranks(const double* v, int n, int* rank) {
    for (int j = 0; j < n; ++j) {
        rank[j] = 0;
        for (int k = 0; k < n; ++k) rank[j] += zh::before_desc(v[k], k, v[j], j) ? 1 : 0;
    }
}
"""


@pytest.fixture(scope="module")
def ranks(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "o.cpp").write_text(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "o.cpp"), "-o", str(d / "o.so")],
                   check=True)
    fn = ctypes.CDLL(str(d / "o.so")).ranks

    def run(v):
        v = np.ascontiguousarray(v, dtype=np.float64)
        out = np.empty(len(v), dtype=np.int32)
        fn(v.ctypes.data_as(ctypes.c_void_p), len(v), out.ctypes.data_as(ctypes.c_void_p))
        return out
    return run


def _check(rank, v):
    v = np.asarray(v, dtype=np.float64)
    key = [(1, 0.0, i) if x != x else (0, -x, i) for i, x in enumerate(v)]
    want = np.empty(len(v), dtype=np.int32)
    want[sorted(range(len(v)), key=lambda i: key[i])] = np.arange(len(v))
    assert np.array_equal(rank, want), v


def test_small_sets_exhaustively(ranks):
    vals = [np.nan, np.inf, -np.inf, 0.0, -0.0, 2.5]
    for n in range(1, 6):
        for v in itertools.product(vals, repeat=n):
            _check(ranks(v), v)


@pytest.mark.parametrize("n", [25, 100])
def test_eigenvalue_counts(ranks, n):
    g = np.random.default_rng(n)
    for nan in (0, 1, n // 2, n):
        v = g.integers(-3, 4, n).astype(np.float64)   # many ties
        v[g.permutation(n)[:nan]] = np.nan
        _check(ranks(v), v)
