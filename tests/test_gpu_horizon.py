"""Inputs that lie further ahead than any delay reaches, met by launches that
were put into a graph before the inputs were there: the trajectory has to be that
of a network that launches every span directly."""
import numpy as np
import pytest
import torch

from paper_2111_04398_amd import mc, workloads

pytestmark = pytest.mark.gpu

D_MAX = 20


def network(scheme, block, npw, spg, stream=None):
    w = workloads.balanced().replace(d_max_steps=D_MAX)
    net = mc.Network(w, stream=stream)
    net.set_launch(scheme=scheme, block=block, neurons_per_wg=npw, steps_per_graph=spg)
    net.reserve(1000)
    return net


def inject_ahead(nets, seed):
    """Strong inputs D_MAX+1 to 126 steps ahead, the same to every network."""
    rng = np.random.default_rng(seed)
    for k in [D_MAX + 1, 126] + [int(x) for x in rng.integers(D_MAX + 1, 127, 20)]:
        i, v = int(rng.integers(0, nets[0].N)), int(rng.integers(20_000_000, 80_000_000))
        for net in nets:
            net.inject(k, i, v)


def assert_equal(a, b, what):
    for x, y in zip(a.spikes(), b.spikes()):
        assert np.array_equal(x, y), what
    for x, y in zip(a.state(), b.state()):
        assert np.array_equal(x.view(np.uint8), y.view(np.uint8)), what
    assert np.array_equal(a.ring(128), b.ring(128)), what


@pytest.mark.parametrize("how", ["inject", "load_state"])
@pytest.mark.parametrize("scheme,block,npw", [(1, 512, 0), (1, 512, 512), (3, 256, 0), (0, 256, 256)])
def test_inputs_ahead_of_a_graph_that_is_already_there(scheme, block, npw, how):
    """The network's own graph of 40 steps has run before the inputs come."""
    net, direct = network(scheme, block, npw, 40), network(scheme, block, npw, 0)
    for n in (net, direct):
        n.simulate(40)
    for seed in (5, 6):
        inject_ahead((net, direct) if how == "inject" else (direct,), seed)
        if how == "load_state":
            net.load_state(direct.save_state())
        for n in (net, direct):
            n.simulate(160)
        assert_equal(net, direct, (scheme, npw, how, seed))


@pytest.mark.parametrize("npw", [0, 512])
def test_inputs_ahead_of_a_graph_that_the_caller_captured(npw):
    """The caller's graph of one mc_simulate_noalloc call is replayed after the inputs came."""
    stream = torch.cuda.Stream()
    net, direct = network(1, 512, npw, 0, stream.cuda_stream), network(1, 512, npw, 0)
    net.simulate_noalloc(40)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        net.simulate_noalloc(40)
    with torch.cuda.stream(stream):
        graph.replay()
    direct.simulate(80)
    inject_ahead((net, direct), 7)
    with torch.cuda.stream(stream):
        for _ in range(4):
            graph.replay()
    direct.simulate(160)
    for x, y in zip(net.spikes() + net.state(), direct.spikes() + direct.state()):
        assert np.array_equal(x.view(np.uint8), y.view(np.uint8))
