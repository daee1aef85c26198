"""GPU parity where a build's rounds stay on the bit-plane table, end on its
last plane, or outgrow it and go on with the byte table: paths whose longest
distances lie around the last plane, alone and hung on a Barabasi-Albert
graph, for every width of a table row (1 to 16 candidate words, whole and
ragged), with one and with four receivers per wave, undirected, directed,
with bit-parallel roots and allocation-free, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1906_12018_amd as pll
import synth
from gpu_util import DEV, assert_labels_equal, build, check_counters, to_dev
from test_gpu_bp import check_bp
from test_gpu_directed import build_dir, check_directed

pytestmark = pytest.mark.gpu

PLANES = 8  # distances a table row holds; round PLANES + 2 needs one more


def tailed(length, n=300):
    """A Barabasi-Albert graph with a path of `length` vertices on its last vertex."""
    g = synth.ba_graph(n, 3, 9)
    rows = np.repeat(np.arange(g.n), np.diff(g.row_ptr).astype(np.int64))
    tail = np.arange(n - 1, n - 1 + length)
    return synth.csr_from_edges(n + length, np.concatenate([rows, tail]), np.concatenate([g.col, tail + 1]))


@pytest.mark.parametrize("flags", [pll.FLAG_VALIDATE, pll.FLAG_VALIDATE | pll.FLAG_PACK4])
@pytest.mark.parametrize("b", [1, 64, 65, 128, 190, 256, 449, 1000])
@pytest.mark.parametrize("length", [PLANES - 2, PLANES, PLANES + 1, PLANES + 2, PLANES + 3, 40])
def test_rounds_around_the_last_plane(length, b, flags):
    for g in (synth.path_graph(length), tailed(length)):
        for order in (synth.degree_order(g), np.random.default_rng(length).permutation(g.n).astype(np.uint32)):
            want = oracle.pll_labels(g, order)
            idx = build(g, order, batch_size=b, flags=flags)
            assert_labels_equal(idx, want, order)
            check_counters(idx, g, order, b, want)
            idx.free()


@pytest.mark.parametrize("b", [64, 130, 1024])
@pytest.mark.parametrize("length", [PLANES + 1, PLANES + 2, 40])
def test_directed_rounds_around_the_last_plane(length, b):
    for g in (synth.directed_path(length + 1), synth.directed_cycle(length + 1), synth.as_digraph(tailed(length))):
        order = synth.degree_order_directed(g)
        idx = build_dir(g, order, batch_size=b)
        check_directed(idx, g, order)
        idx.free()


@pytest.mark.parametrize("length", [PLANES + 1, 40])
def test_bit_parallel_rounds_around_the_last_plane(length):
    g = tailed(length)
    order = synth.degree_order(g)
    idx = build(g, order, batch_size=128, bp_roots=3)
    check_bp(idx, g, order, 3)
    idx.free()


@pytest.mark.parametrize("b", [64, 256])
@pytest.mark.parametrize("length", [PLANES + 1, PLANES + 2, 40])
def test_noalloc_rounds_around_the_last_plane(length, b):
    g = tailed(length)
    order = synth.degree_order(g)
    want = oracle.pll_labels(g, order)
    rp, cl, od = to_dev(g, order)
    off = torch.zeros(g.n + 1, dtype=torch.int64, device=DEV)
    hubs = torch.zeros(want.total, dtype=torch.int32, device=DEV)
    dists = torch.zeros(want.total, dtype=torch.uint8, device=DEV)
    assert pll.build_labels_noalloc(rp, cl, od, off, hubs, dists, batch_size=b) == want.total
    assert np.array_equal(off.cpu().numpy().view(np.uint64), want.offsets)
    assert np.array_equal(hubs.cpu().numpy().view(np.uint32), want.hubs_as_ids(order))
    assert np.array_equal(dists.cpu().numpy(), want.dist)


@pytest.mark.parametrize("flags", [0, pll.FLAG_RECHECK])
@pytest.mark.parametrize("b,max_gang", [(64, 1), (190, 3), (1024, 16)])
def test_many_graphs_around_the_last_plane(b, max_gang, flags):
    # graphs that stay on the planes beside graphs that leave them, and rows
    # long enough to be pushed as items of their own
    graphs = [tailed(k) for k in (1, PLANES, PLANES + 1, PLANES + 2, 40)] + [
        synth.path_graph(200), synth.star_graph(3000), synth.ba_graph(2500, 4, 3), synth.disjoint_union(
            synth.star_graph(2100), synth.path_graph(30))]
    orders = [synth.degree_order(g) for g in graphs]
    idxs = pll.build_labels_batched([to_dev(g, o) for g, o in zip(graphs, orders)], batch_size=b, flags=flags,
                                    gang_scale=1000, max_gang=max_gang)
    for g, o, idx in zip(graphs, orders, idxs):
        want = oracle.pll_labels(g, o)
        assert_labels_equal(idx, want, o)
        check_counters(idx, g, o, b, want)
        idx.free()
