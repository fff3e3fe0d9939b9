"""Device memory of a network: what happens when it runs out, and what goes back."""
import numpy as np
import pytest
import torch

from paper_2111_04398_amd import mc, workloads
from test_oracle_dynamics import lone_neuron

pytestmark = pytest.mark.gpu


class Hooks:
    """Allocator hooks on torch's caching allocator that refuse the sizes in `refuse`."""

    def __init__(self):
        self.live, self.refuse, self.refused = {}, set(), 0

    def alloc(self, nbytes):
        if nbytes in self.refuse:
            self.refused += 1
            return None
        p = torch.cuda.caching_allocator_alloc(nbytes)
        self.live[p] = nbytes
        return p

    def free(self, ptr):
        del self.live[ptr]
        torch.cuda.caching_allocator_delete(ptr)

    def network(self, w):
        return mc.Network(w, allocator=(lambda nbytes: self.alloc(nbytes), lambda ptr: self.free(ptr)))


def same_spikes(a, b):
    (s0, i0), (s1, i1) = a.spikes(), b.spikes()
    return len(s0) > 0 and np.array_equal(s0, s1) and np.array_equal(i0, i1)


@pytest.mark.parametrize("scheme,block,npw", [(0, 256, 256), (2, 256, 256), (3, 256, 0)])
def test_without_memory_for_the_packed_rows_the_network_keeps_its_launch(scheme, block, npw):
    """The persistent scheme's copy of the store (8 B per synapse) does not fit: mc_set_launch says so, and
    the network goes on with the launch it had; the autotuner passes over the scheme."""
    w = workloads.balanced()
    hooks = Hooks()
    net, twin = hooks.network(w), mc.Network(w)
    for n in (net, twin):
        n.set_launch(scheme=scheme, block=block, neurons_per_wg=npw, steps_per_graph=100)
        n.simulate(150)
    hooks.refuse = {8 * net.M}
    before = dict(hooks.live)
    with pytest.raises(mc.MCError) as e:
        net.set_launch(scheme=1, block=512, neurons_per_wg=0, steps_per_graph=100)
    assert e.value.code == -3 and hooks.refused >= 1
    assert sorted(hooks.live.values()) == sorted(before.values())
    for n in (net, twin):
        n.simulate(150)
    assert same_spikes(net, twin) and net.counters()["events"] == twin.counters()["events"]
    net.tune(200)
    for n in (net, twin):
        n.simulate(150)
    assert same_spikes(net, twin)
    net.close()
    assert not hooks.live


def test_packed_rows_are_kept_where_they_are_used_and_go_back_elsewhere():
    w = workloads.balanced()
    hooks = Hooks()
    net, twin = hooks.network(w), mc.Network(w)
    rows = 8 * net.M

    def held():
        return sum(1 for b in hooks.live.values() if b == rows)

    for scheme, npw, want in ((1, 0, 1), (1, 64, 1), (0, 256, 0), (1, 64, 1), (3, 0, 0), (1, 0, 1), (2, 256, 0)):
        net.set_launch(scheme=scheme, block=256, neurons_per_wg=npw, steps_per_graph=100)
        assert held() == want, (scheme, npw)
        for n in (net, twin):
            n.simulate(120)
    assert same_spikes(net, twin)


def test_buffers_of_a_long_read_back_go_back():
    """17 million spikes at once (a burst of a million neurons every 68 steps): 100 MB of scratch."""
    n = 1_000_000
    hooks = Hooks()
    net = hooks.network(lone_neuron(i_e=1000.0).replace(pop_size=[n]))
    net.set_launch(scheme=0, block=256, neurons_per_wg=1024, steps_per_graph=0)
    net.reserve(1136)
    before = sorted(hooks.live.values())
    net.simulate(1136)
    s, i = net.spikes()
    assert np.array_equal(s, np.repeat(np.arange(47, 1136, 68, dtype=np.int32), n)) and np.array_equal(i[-n:], i[:n])
    assert np.array_equal(i[:n], np.arange(n, dtype=np.int32))
    assert sorted(hooks.live.values()) == before


@pytest.mark.parametrize("mode", [mc.ADJ_INPUT_RECORD, mc.ADJ_INPUT_REPLAY])
def test_buffers_of_an_adjoint_that_fails_go_back_after_its_kernels(mode):
    """No memory for the reverse pass's lists, the last allocation of the call: forward and recompute are queued
    by then, and end before any buffer goes back to the allocator."""
    w = workloads.microcircuit(scale=0.05)
    hooks, idle = Hooks(), []
    net = hooks.network(w)
    net.set_launch(scheme=1, block=512, neurons_per_wg=0, steps_per_graph=0)
    net.reserve(4096)
    stream = torch.cuda.ExternalStream(net.stream())
    free, alloc = hooks.free, hooks.alloc
    sizes = []
    hooks.alloc = lambda nbytes: sizes.append(nbytes) or alloc(nbytes)
    hooks.free = lambda ptr: (idle.append(stream.query()), free(ptr))
    fresh = net.save_state()
    grad = torch.empty(net.M, dtype=torch.float64, device="cuda")

    def adjoint():
        net.load_state(fresh)
        return net.adjoint(2000, 2000, -58.0, False, grad.data_ptr(), input_mode=mode)

    loss = adjoint()
    assert adjoint() == loss
    want = grad.clone()
    hooks.refuse = {sizes[-1]}
    del idle[:]
    with pytest.raises(mc.MCError) as e:
        adjoint()
    assert e.value.code == -3 and hooks.refused == 1 and len(idle) >= 8 and all(idle)
    hooks.refuse = set()
    assert adjoint() == loss and torch.equal(grad, want)
