"""The adjoint's gather by target ranges, at the sizes around its rule.

Networks whose LI values of 60 steps exceed 4 MiB (more than 8,738 neurons)
take the gather that splits every row into eight target ranges.  Every
synapse's terms are added in the same order either way, so gradient and loss
have to be the oracle's to the bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2111_04398_amd import mc, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pops", [[8000, 700], [8000, 740], [8000, 801], [11001, 2999]])
@pytest.mark.parametrize("fp32", [False, True])
def test_gather_matches_oracle_on_both_sides_of_the_rule(pops, fp32):
    w = workloads.balanced(seed=3).replace(pop_size=pops, conn=[[60.0, 15.0], [60.0, 0.0]], k_ext=[1500.0, 1500.0])
    S, K = 230, 50
    y_star = -58.0 - (-65.0)
    ol, og = oracle.Oracle(w.to_dict()).adjoint(S, y_star, fp32=fp32)
    assert np.count_nonzero(og) > 1000
    net = mc.Network(w)
    fresh = net.save_state()
    dt = torch.float32 if fp32 else torch.float64
    for rep in range(2):                       # the second pass finds the range table made
        if rep:
            net.load_state(fresh)
        g = torch.empty(net.M, dtype=dt, device="cuda")
        loss = net.adjoint(S, K, -58.0, fp32, g.data_ptr())
        assert abs(loss - ol) <= 1e-12 * abs(ol)
        bits = np.uint32 if fp32 else np.uint64
        assert np.array_equal(g.cpu().numpy().view(bits), og.view(bits))
