"""GPU parity of builds whose batches are queued ahead of the host, where a
queue halts: batches that need more rounds than the one before, rows long
enough for a launch of their own met by a later batch, rounds that outgrow
the planes behind a queue, and a last, ragged batch, against the oracle
(labels and Algorithm 4's counters)."""
import numpy as np
import pytest

import oracle
import paper_1906_12018_amd as pll
import synth
from gpu_util import assert_labels_equal, build, check_counters
from test_gpu_bp import check_bp
from test_gpu_directed import build_dir, check_directed
from test_gpu_weighted import build_w, check_weighted

pytestmark = pytest.mark.gpu


def graphs():
    star = synth.star_graph(2600)
    ba = synth.ba_graph(1800, 3, 4)
    tree = synth.random_tree(900, 7)
    comb = synth.disjoint_union(*[synth.path_graph(k) for k in (2, 9, 4, 30, 3, 12, 60, 5, 8)] * 6)
    return [star, ba, tree, comb, synth.disjoint_union(ba, star, synth.path_graph(70)),
            synth.disjoint_union(*[synth.star_graph(1100 + k) for k in range(3)])]


@pytest.mark.parametrize("b", [16, 61, 128])
@pytest.mark.parametrize("seed", [0, 1, 2])
@pytest.mark.parametrize("gi", range(len(graphs())))
def test_queues_that_halt(gi, seed, b):
    g = graphs()[gi]
    order = synth.degree_order(g) if seed == 0 else np.random.default_rng(seed).permutation(g.n).astype(np.uint32)
    want = oracle.pll_labels(g, order)
    idx = build(g, order, batch_size=b, flags=0)
    assert_labels_equal(idx, want, order)
    check_counters(idx, g, order, b, want)
    idx.free()


def digraphs():
    star = synth.star_graph(2200)
    out_star = synth.DiGraph(n=2200, row_ptr=np.concatenate([[0], np.full(2200, 2199)]).astype(np.uint64),
                             col=np.arange(1, 2200, dtype=np.uint32))
    return [synth.as_digraph(star), out_star, synth.reverse_digraph(out_star), synth.rmat_digraph(10, 5, seed=3),
            synth.directed_cycle(60), synth.gnp_digraph(300, 0.006, 4),
            synth.as_digraph(synth.disjoint_union(synth.ba_graph(600, 2, 5), synth.star_graph(1200)))]


def directed_rounds(g, order, b):
    """Lockstep rounds of the two sides by the labels: a batch runs one round
    more than the largest distance of the entries its roots gained."""
    lin, lout = oracle.pll_labels_directed(g, order)
    rounds = 0
    for ib in range(0, g.n, b):
        far = 0
        for lab in (lin, lout):
            mine = (lab.hub_rank >= ib) & (lab.hub_rank < ib + b)
            far = max(far, int(lab.dist[mine].max(initial=0)))
        rounds += 1 + far
    return rounds


@pytest.mark.parametrize("b", [16, 61, 128])
@pytest.mark.parametrize("seed", [0, 1])
@pytest.mark.parametrize("gi", range(len(digraphs())))
def test_directed_queues_that_halt(gi, seed, b):
    g = digraphs()[gi]
    order = (synth.degree_order_directed(g) if seed == 0
             else np.random.default_rng(seed).permutation(g.n).astype(np.uint32))
    idx = build_dir(g, order, batch_size=b)
    check_directed(idx, g, order)
    assert idx.info()["rounds"] == directed_rounds(g, order, b)
    idx.free()


@pytest.mark.parametrize("n,b", [(1500, 256), (4000, 1024)])
def test_weighted_rounds_gathered_and_pushed(n, b):
    # dense first batches gather, later ones push; rows of several gather
    # segments beside short ones
    g = synth.with_weights(synth.disjoint_union(synth.ba_graph(n, 6, 3), synth.star_graph(700)))
    order = synth.degree_order(g)
    idx = build_w(g, order, batch_size=b)
    check_weighted(idx, g, order)
    idx.free()


@pytest.mark.parametrize("b", [16, 100])
def test_bit_parallel_queues(b):
    g = synth.disjoint_union(synth.ba_graph(1500, 3, 8), synth.star_graph(1300), synth.path_graph(40))
    order = np.random.default_rng(5).permutation(g.n).astype(np.uint32)
    idx = build(g, order, batch_size=b, bp_roots=4)
    check_bp(idx, g, order, 4)
    idx.free()


def test_queue_meets_a_small_arena():
    # the arena fills while batches are queued: the build still reports it
    g = synth.ba_graph(3000, 4, 2)
    order = synth.degree_order(g)
    need = oracle.pll_labels(g, order).total
    with pytest.raises(pll.PllError) as e:
        build(g, order, batch_size=64, arena_entries=32 * g.n + need // 4)
    assert e.value.status == pll.PLL_ENOSPC
