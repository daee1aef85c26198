"""Directed batches queued ahead of the host check four receivers per wave
where both sides together expect the receivers for it, as the rounds that the
host launches do.  A packed scan takes 16 label entries a step, a whole wave
64, so the packed form shows in the entries it reads before it stops."""
import numpy as np
import pytest
import torch

import paper_1906_12018_amd as pll
import synth
from gpu_util import DEV
from test_gpu_directed import build_dir, check_directed

pytestmark = pytest.mark.gpu


def entries_read(g, order, b, flags):
    rp, cl = pll.graph_to_device(g, DEV)
    od = torch.from_numpy(np.ascontiguousarray(order).view(np.int32)).to(DEV)
    idx = pll.build_labels_directed(rp, cl, od, batch_size=b, flags=flags)
    info = idx.info()
    idx.free()
    return info["check_entries_read"], info["candidates"], info["rounds"]


def test_queued_rounds_of_many_receivers_pack():
    # 8,192 vertices: the first batch is queued with every vertex expected on both sides
    g = synth.rmat_digraph(13, 8, seed=3)
    order = synth.degree_order_directed(g)
    queued = entries_read(g, order, 1024, 0)
    by_round = entries_read(g, order, 1024, pll.FLAG_PROFILE)  # the host launches every round; its first is not packed
    assert queued[1:] == by_round[1:]
    assert queued[0] < by_round[0]


@pytest.mark.parametrize("scale,b", [(12, 256), (13, 1000)])
def test_labels_of_packed_queued_rounds(scale, b):
    g = synth.rmat_digraph(scale, 6, seed=scale)
    order = synth.degree_order_directed(g)
    idx = build_dir(g, order, batch_size=b, flags=0)
    check_directed(idx, g, order)
    idx.free()
