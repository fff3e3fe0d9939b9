"""The persistent scheme's id queue with little room (the MC_PERSIST_LIST_CAP
hook, honoured by the launches that mc_profile_phases makes): bursts bring far
more ids than it holds, so its poller waits for deliveries and its slots are used
again and again.  The trajectory stays the oracle's."""
import pytest

import oracle
from paper_2111_04398_amd import mc, workloads
from test_gpu_parity import assert_same

pytestmark = pytest.mark.gpu


# four targets per workgroup: every burst comes as short records of four spikes, polled four (250
# workgroups) or eight (500) per lane; 20 and 200 targets: as bitmaps
@pytest.mark.parametrize("cap", [1, 33, 1000])
@pytest.mark.parametrize("pops,block,npw", [([800, 200], 512, 4), ([1600, 400], 256, 4), ([4000, 1000], 512, 0),
                                            ([4000, 1000], 256, 200)])
def test_bursts_through_a_small_queue(pops, block, npw, cap, monkeypatch):
    w = workloads.balanced().replace(name="bursts", i_e=1.0e5, pop_size=pops)
    monkeypatch.setenv("MC_PERSIST_LIST_CAP", str(cap))
    net, o = mc.Network(w), oracle.Oracle(w.to_dict())
    net.set_launch(scheme=1, block=block, neurons_per_wg=npw, steps_per_graph=0)
    net.profile_phases(150)
    o.run(150)
    assert len(o.raster()[0]) == sum(pops) * 8
    assert_same(net, o, what=f"{pops}, {npw} targets, room for {cap}")
