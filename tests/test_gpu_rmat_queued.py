"""R-MAT scale 16 as the benchmark's timed steps build it (b = 1024, no flags:
small rounds queued ahead of the host), the labels and Algorithm 4's counters
against the oracle."""
import pytest

import oracle
import synth
from gpu_util import assert_labels_equal, build, check_counters

pytestmark = pytest.mark.gpu


def test_rmat16_queued_build():
    g = synth.rmat_graph(16)
    order = synth.degree_order(g)
    want = oracle.pll_labels(g, order)
    idx = build(g, order, batch_size=1024, flags=0)
    assert_labels_equal(idx, want, order)
    info = check_counters(idx, g, order, 1024, want)
    assert info["batches"] == 64
    idx.free()
