"""Exact queries at the sizes where a call's split changes: one pair, the
edges of a wave's group of pairs, and the last call that takes a wave per pair
and the first that does not, on an index with short lists, one with
bit-parallel roots and a directed one, against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import build, gpu_query
from test_gpu_directed import build_dir

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 63, 64, 65, 1000, 32767, 32768, 32769, 65537, 140000]


def indexes():
    g = synth.ba_graph(1500, 2, 5)
    order = synth.degree_order(g)
    lab = oracle.pll_labels(g, order)
    yield g, build(g, order), lambda u, v: oracle.query(lab, u, v)
    blab, bp = oracle.pll_labels_bp(g, order, 16)
    yield g, build(g, order, bp_roots=16), lambda u, v: oracle.query_bp(blab, bp, u, v)
    d = synth.rmat_digraph(10, 6, seed=5)
    order = synth.degree_order_directed(d)
    lin, lout = oracle.pll_labels_directed(d, order)
    yield d, build_dir(d, order), lambda u, v: oracle.query_directed(lin, lout, u, v)


def test_calls_of_few_pairs():
    for g, idx, want in indexes():
        u, v = synth.query_pairs(g.n + 3, max(COUNTS), seed=11)  # some ids are out of range
        ok = (u < g.n) & (v < g.n)
        exact = np.full(u.size, oracle.DIST_INF, dtype=np.uint32)
        exact[ok] = want(u[ok], v[ok])
        for count in COUNTS:
            assert np.array_equal(gpu_query(idx, u[:count], v[:count]), exact[:count]), count
        idx.free()
