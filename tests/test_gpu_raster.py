"""The raster's read-back (ordered on the device) against the oracle, at the
edges of its ways: no spike, one workgroup's sort up to 2,048 spikes, beyond
that a step's spikes by rank (up to 256) and through the id bitmap (one and
several passes of 2^18 ids)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2111_04398_amd import mc, workloads
from test_gpu_parity import assert_same
from test_oracle_dynamics import lone_neuron

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme,block,npw", [(0, 256, 256), (1, 512, 0), (3, 256, 0)])
@pytest.mark.parametrize("steps", [1, 2, 300])
def test_read_back_after_every_span(scheme, block, npw, steps):
    """Spans of 0 to ~2,000 spikes and of several thousand, read after each and all at once."""
    w = workloads.balanced()
    net, whole, o = mc.Network(w), mc.Network(w), oracle.Oracle(w.to_dict())
    for n in (net, whole):
        n.set_launch(scheme=scheme, block=block, neurons_per_wg=npw, steps_per_graph=100)
    got = []
    for k in range(4):
        net.simulate(steps)
        got.append(net.spikes(k * steps, (k + 1) * steps))
    whole.simulate(4 * steps)
    o.run(4 * steps)
    os_, oi = o.raster()
    assert np.array_equal(np.concatenate([g[0] for g in got]), os_)
    assert np.array_equal(np.concatenate([g[1] for g in got]), oi)
    assert_same(whole, o, ring_depth=4, what="one read-back")


@pytest.mark.parametrize("n", [255, 2048, 2049, 300000])
def test_every_neuron_fires_at_once(n):
    """All neurons of an unconnected population fire in the same steps: total and per-step
    counts on both sides of the limits, ids beyond one bitmap pass."""
    w = lone_neuron(i_e=1000.0).replace(pop_size=[n])
    net = mc.Network(w)
    net.set_launch(scheme=0, block=256, neurons_per_wg=256, steps_per_graph=0)
    net.simulate(200)
    s, i = net.spikes()
    one = mc.Network(lone_neuron(i_e=1000.0))
    one.simulate(200)
    ref = one.spikes()[0]
    assert len(ref) >= 1 and len(s) == n * len(ref)
    assert np.array_equal(s, np.repeat(ref, n)) and np.array_equal(i, np.tile(np.arange(n, dtype=np.int32), len(ref)))


def captured_spans(net, stream, steps):
    """A graph that the caller captured, of one mc_simulate_noalloc call on the network's stream."""
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        net.simulate_noalloc(steps)
    return graph


@pytest.mark.parametrize("npw", [0, 256])
def test_read_back_after_a_callers_graph_ran_more_steps_than_the_host_counted(npw):
    """A program that captures a span and replays it: every replay's spikes come back, once, also
    when none has been counted since the last read-back, and beyond 2,048 spikes."""
    w = workloads.balanced()
    stream = torch.cuda.Stream()
    net, o = mc.Network(w, stream=stream.cuda_stream), oracle.Oracle(w.to_dict())
    net.set_launch(scheme=1, block=512, neurons_per_wg=npw, steps_per_graph=0)
    net.reserve(4000)
    net.simulate_noalloc(100)
    o.run(100)
    assert len(net.spikes()[0]) == len(o.raster()[0])
    graph = captured_spans(net, stream, 100)
    for replays in (1, 1, 4, 1, 9):
        for _ in range(replays):
            with torch.cuda.stream(stream):
                graph.replay()
        before = len(o.raster()[0])
        o.run(100 * replays)
        (s, i), (os_, oi) = net.spikes(), o.raster()
        assert len(os_) > before and np.array_equal(s, os_) and np.array_equal(i, oi), replays
    assert len(net.spikes()[0]) == len(o.raster()[0])


@pytest.mark.parametrize("n,steps", [(2047, 48), (2048, 48), (2049, 48), (255, 700), (256, 700), (257, 700),
                                     (2**18, 48), (2**18 + 1, 48)])
def test_read_back_at_the_limits_of_its_ways(n, steps):
    """One burst of 2,047 to 2,049 spikes in all (one workgroup, or the long way); bursts of 255 to
    257 spikes of which the long way reads more than 2,048 (by rank, or through the bitmap); a burst
    on both sides of one bitmap pass."""
    w = lone_neuron(i_e=1000.0)
    o = oracle.Oracle(w.to_dict())
    o.run(steps)
    ref = o.raster()[0]
    assert len(ref) == 1 if steps == 48 else len(ref) * n > 2048
    net = mc.Network(w.replace(pop_size=[n]))
    net.set_launch(scheme=0, block=256, neurons_per_wg=256, steps_per_graph=0)
    net.simulate(steps)
    s, i = net.spikes()
    assert np.array_equal(s, np.repeat(ref, n)) and np.array_equal(i, np.tile(np.arange(n, dtype=np.int32), len(ref)))


def test_read_back_of_more_segments_than_one_workgroup_sums():
    """5,000 segments: always the long way, without and with spikes."""
    w = lone_neuron(i_e=1000.0).replace(pop_size=[20000])
    net = mc.Network(w)
    net.set_launch(scheme=0, block=64, neurons_per_wg=4, steps_per_graph=0)
    net.simulate(10)
    assert len(net.spikes()[0]) == 0
    net.simulate(38)
    s, i = net.spikes()
    assert np.array_equal(s, np.full(20000, 47, np.int32)) and np.array_equal(i, np.arange(20000, dtype=np.int32))
