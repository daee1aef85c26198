"""The serving loop's copy threads (csrc/pll_copy.h), compiled here for the
host: every byte arrives, and small requests are handed out in parts of the
same size as large ones."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import paper_1906_12018_amd

CSRC = os.path.join(os.path.dirname(os.path.abspath(paper_1906_12018_amd.__file__)), "csrc")

SHIM = r"""
#include "pll_copy.h"
extern "C" void* pool(unsigned helpers) {
    auto* p = new pll::CopyPool;
    p->start(helpers);
    return p;
}
extern "C" void drop(void* p) { delete static_cast<pll::CopyPool*>(p); }
extern "C" unsigned long long copy(void* p, char* dst, const char* src, const unsigned long long* at, unsigned n) {
    auto* c = static_cast<pll::CopyPool*>(p);
    for (unsigned i = 0; i < n; ++i) c->add(dst + at[i], src + at[i], at[i + 1] - at[i]);
    return c->run();
}
extern "C" unsigned long long part() { return pll::CopyPool::kPart; }
"""


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    d = tmp_path_factory.mktemp("copy")
    (d / "copy.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-shared", "-fPIC", "-I", CSRC, "-o",
                           str(d / "libcopy.so"), str(d / "copy.cpp")])
    lib = ctypes.CDLL(str(d / "libcopy.so"))
    lib.pool.restype = ctypes.c_void_p
    lib.drop.argtypes = [ctypes.c_void_p]
    lib.copy.argtypes = [ctypes.c_void_p] * 4 + [ctypes.c_uint]
    lib.copy.restype = lib.part.restype = ctypes.c_ulonglong
    return lib


def run(so, pool, sizes, seed):
    at = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    src = np.random.default_rng(seed).integers(0, 256, int(at[-1]), dtype=np.uint8)
    dst = np.zeros_like(src)
    parts = so.copy(pool, dst.ctypes.data, src.ctypes.data, at.ctypes.data, len(sizes))
    assert np.array_equal(dst, src)
    return parts


@pytest.mark.parametrize("helpers", [0, 1, 6])
def test_copies_are_whole_and_parts_even(so, helpers):
    pool = so.pool(helpers)
    k = so.part()
    rng = np.random.default_rng(helpers)
    for seed, sizes in enumerate([[], [0], [1], [k - 1], [k], [k + 1], [8 * k + 3, 0, 5], [800] * 8000,
                                  rng.integers(0, 3 * k, 60).tolist(), rng.integers(0, 2000, 5000).tolist()]):
        for _ in range(3):
            parts = run(so, pool, sizes, seed)
            # a part holds at least kPart bytes, but for the last and for the ends of large copies
            assert parts <= sum(sizes) / k + sum(s > k for s in sizes) + 1
    so.drop(pool)


def test_thousands_of_small_copies_make_few_parts(so):
    pool = so.pool(6)
    k = so.part()
    assert run(so, pool, [800] * 4000, 1) == -(-800 * 4000 // (-(-k // 800) * 800))
    so.drop(pool)
