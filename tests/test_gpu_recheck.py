"""The recheck's scan reads only table words that can decide: an entry at
distance d covers no candidate at d or below.  In a complete graph every entry
is at distance 1, so a build with the recheck reads no table word at all."""
import numpy as np
import pytest

import oracle
import paper_1906_12018_amd as pll
import synth
from gpu_util import assert_labels_equal, build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, pll.FLAG_RELAXED, pll.FLAG_PERSISTENT])
@pytest.mark.parametrize("n,b", [(70, 64), (150, 128), (300, 1024)])
def test_recheck_of_equal_distances_reads_no_table(n, b, flags):
    g = synth.complete_graph(n)
    order = np.random.default_rng(n).permutation(n).astype(np.uint32)
    idx = build(g, order, batch_size=b, flags=pll.FLAG_RECHECK | flags)
    assert_labels_equal(idx, oracle.pll_labels(g, order), order)
    info = idx.info()
    assert info["recheck_removed"] == 0
    assert info["check_table_reads"] == 0
    idx.free()


def test_recheck_of_two_distances():
    # a cycle a - b - x - v - a: b reaches v over x at distance 2, which a covers
    g = synth.csr_from_edges(4, np.array([0, 1, 2, 3]), np.array([1, 2, 3, 0]))
    order = np.arange(4, dtype=np.uint32)
    idx = build(g, order, batch_size=64, flags=pll.FLAG_RECHECK | pll.FLAG_RELAXED)
    assert_labels_equal(idx, oracle.pll_labels(g, order), order)
    assert idx.info()["recheck_removed"] == 1
    idx.free()
