"""Persistent launches that leave room on the GPU for another network's.

The workgroups of a persistent launch wait for one another, so two launches that
overlap both have to fit whole.  A small network's workgroups take no more
threads than its launch configuration names: two networks on two streams run
beside each other.  With as few wavefronts as that, one has several roles."""
import numpy as np
import pytest

import oracle
from paper_2111_04398_amd import mc, workloads
from test_gpu_parity import assert_same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [(256, 256), (512, 256)])
def test_two_networks_run_beside_each_other(blocks):
    """Both have nearly as many workgroups as the GPU has compute units, and 0.4 s of model time
    each in one launch."""
    works = [workloads.balanced(seed=s) for s in (3, 4)]
    nets = [mc.Network(w) for w in works]
    for net, block in zip(nets, blocks):
        net.set_launch(scheme=1, block=block, neurons_per_wg=0, steps_per_graph=0)
        assert net.persist_shape()["workgroups"] > 240
        net.reserve(8000)
    for _ in range(2):
        for net in nets:
            net.simulate(4000)
    for net, w in zip(nets, works):
        o = oracle.Oracle(w.to_dict())
        o.run(8000)
        assert_same(net, o, what=f"beside another, blocks {blocks}")


@pytest.mark.parametrize("block,npw", [(64, 0), (64, 64), (128, 0), (128, 128), (192, 100), (320, 0)])
def test_few_wavefronts(block, npw):
    """One wavefront that updates, polls and delivers; two of which the poller updates too; and up to five."""
    w = workloads.balanced().replace(pop_size=[1600, 400])
    net, o = mc.Network(w), oracle.Oracle(w.to_dict())
    net.set_launch(scheme=1, block=block, neurons_per_wg=npw, steps_per_graph=300)
    assert net.persist_shape()["lds_steps"] == 102
    net.simulate(1000)
    o.run(1000)
    assert len(o.raster()[0]) > 500
    assert_same(net, o, what=f"block {block}, {npw} targets")
