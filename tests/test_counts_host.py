"""The counts of the phases (csrc/pll_stats.h), compiled here for the host: a
lane keeps 32 bits of a round, and a kernel that runs many rounds sums them in
64 bits, so its totals do not wrap."""
import ctypes
import os
import subprocess

import numpy as np

import paper_1906_12018_amd

CSRC = os.path.join(os.path.dirname(os.path.abspath(paper_1906_12018_amd.__file__)), "csrc")

SHIM = r"""
#include "pll_stats.h"
// `rounds` rounds that count `per` table quarters and entries each
extern "C" void run(unsigned rounds, unsigned per, unsigned long long* tot) {
    pll::PhaseStats st;
    for (unsigned r = 0; r < rounds; ++r) {
        st.table += per;
        st.read += per;
        st.cand += 1;
        st.cost_pos += 5ull * per;
        unsigned long long v[pll::kCounts] = {};
        pll::take_counts(st, v);
        for (int k = 0; k < pll::kCounts; ++k) tot[k] += v[k];
    }
    tot[pll::kCountRemoved] += st.table + st.read;  // nothing stays behind
}
extern "C" int at(int which) {
    const int k[4] = {pll::kCountTable, pll::kCountRead, pll::kCountCand, pll::kCountPos};
    return which < 4 ? k[which] : (int)pll::kCounts;
}
"""


def test_counts_of_many_rounds_do_not_wrap(tmp_path):
    src, lib = tmp_path / "counts.cpp", tmp_path / "libcounts.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib),
                           str(src)])
    so = ctypes.CDLL(str(lib))
    tot = np.zeros(so.at(4), dtype=np.uint64)
    rounds, per = 9, 0xF0000000
    so.run(ctypes.c_uint(rounds), ctypes.c_uint(per), tot.ctypes.data_as(ctypes.c_void_p))
    assert [int(tot[so.at(k)]) for k in range(4)] == [rounds * per, rounds * per, rounds, rounds * per * 5]
    assert int(tot.sum()) == 7 * rounds * per + rounds
