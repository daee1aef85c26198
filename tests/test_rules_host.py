"""The rules that choose a query call's lanes (csrc/pll_rules.h), compiled here
for the host and held against measured times of both sides of each line."""
import ctypes
import os
import subprocess

import pytest

import paper_1906_12018_amd

CSRC = os.path.join(os.path.dirname(os.path.abspath(paper_1906_12018_amd.__file__)), "csrc")

SHIM = r"""
#include "pll_rules.h"
extern "C" unsigned lanes(uint64_t n, uint64_t entries, uint64_t longest, uint64_t roots) {
    return pll::query_lanes(pll::LabelShape{n, entries, longest, roots});
}
extern "C" unsigned long long small_call(uint64_t n, uint64_t entries, uint64_t longest, uint64_t roots) {
    return pll::query_small_call(pll::LabelShape{n, entries, longest, roots});
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o",
                           str(d / "librules.so"), str(d / "rules.cpp")])
    so = ctypes.CDLL(str(d / "librules.so"))
    so.lanes.argtypes = so.small_call.argtypes = [ctypes.c_uint64] * 4
    so.small_call.restype = ctypes.c_ulonglong
    return so


# n, mean, longest label, roots; us of 4,000,000 random pairs with 8, 16, 32 and 64 lanes (R-MAT, Barabasi-Albert, torus)
MEASURED = [
    (131072, 58.4, 825, 4, [1467, 1309, 1318, 1168]),
    (262144, 49.8, 817, 16, [1327, 1169, 1235, 1107]),
    (400000, 32.3, 440, 64, [1587, 1450, 1446, 1176]),
    (600000, 43.4, 612, 64, [1931, 1718, 1638, 1209]),
    (65536, 57.8, 794, 1, [1422, 1264, 1281, 1203]),
    (65536, 38.2, 612, 4, [968, 927, 1064, 1130]),
    (131072, 29.8, 422, 16, [857, 806, 1004, 1064]),
    (10000, 47.2, 191, 4, [684, 708, 885, 1550]),
    (20000, 53.2, 262, 16, [933, 893, 1065, 1861]),
    (50000, 41.4, 225, 64, [1511, 1462, 1534, 1884]),
    (4096, 62.8, 137, 16, [794, 808, 921, 1594]),
    (65536, 17.0, 236, 16, [561, 584, 879, 1016]),
]


@pytest.mark.parametrize("n,mean,longest,roots,us", MEASURED)
def test_lanes_with_roots_are_near_the_fastest(rules, n, mean, longest, roots, us):
    lanes = rules.lanes(n, int(n * mean), longest, roots)
    assert us[[8, 16, 32, 64].index(lanes)] <= 1.1 * min(us)


def test_lanes_without_roots(rules):
    for mean, lanes in ((0, 4), (16, 4), (17, 8), (31, 8), (32, 64), (500, 64)):
        for longest in (mean, 100 * mean):
            assert rules.lanes(1000, 1000 * mean, longest, 0) == lanes
            assert rules.small_call(1000000, 1000000 * mean, longest, 0) == 32768
    assert rules.lanes(0, 0, 0, 0) == 4


@pytest.mark.parametrize("n,mean,longest,roots,pairs", [
    (200000, 15, 49, 4, 24576), (50000, 3, 12, 16, 24576), (50000, 3, 12, 64, 32768), (20000, 3, 11, 4, 32768),
    (50000, 40, 185, 16, 32768), (100000, 26, 336, 16, 32768)])
def test_small_calls(rules, n, mean, longest, roots, pairs):
    assert rules.small_call(n, n * mean, longest, roots) == pairs
