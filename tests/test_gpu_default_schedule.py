"""The schedule a new handle starts with, by size, delays and inboxes."""
import pytest

from paper_1902_08410_amd import workloads as W

pytestmark = pytest.mark.gpu

FUSED, SPLIT = 0, 1
J = dict(J_mean=[0.1, -0.4], J_sd=[0.0, 0.0])
CASES = {
    "default": (FUSED, dict()),
    "no_synapses": (FUSED, dict(K_out=0)),
    "plastic": (SPLIT, W.stdp()),
    # what spikes send over one step: K_out / delays of at most 64, or more
    "one_delay": (SPLIT, dict(d_max=1)), "delays_10": (SPLIT, dict(d_max=10)),
    "delays_15": (SPLIT, dict(d_max=15)), "delays_16": (FUSED, dict(d_max=16)),
    "one_delay_of_2": (FUSED, dict(d_min=2, d_max=2)),
    "one_delay_64_synapses": (FUSED, dict(d_max=1, K_out=64)),
    # no inboxes: by request, or for more than 128 slots
    "no_inboxes": (SPLIT, dict(queue_cap=-1)), "slots_150": (SPLIT, dict(d_min=100, d_max=149)),
    "no_inboxes_256": (FUSED, dict(queue_cap=-1, K_out=256)),
    # 1.02 M neurons: few synapses per delay, or more
    "few_1.02M": (SPLIT, dict(grid_w=16, grid_h=32, K=2000, K_out=160, **J)),
    "more_1.02M": (FUSED, dict(grid_w=16, grid_h=32, K=2000, K_out=161, **J)),
    "below_2M": (FUSED, dict(grid_w=31, grid_h=32, K=2000, K_out=161, **J)),
    "above_2M": (SPLIT, dict(grid_w=32, grid_h=32, K=2000, K_out=161, **J)),
    "few_0.99M": (FUSED, dict(grid_w=16, grid_h=31, K=2000, K_out=160, **J)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_default_schedule(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_08410_amd import dpsnn
    want, over = CASES[case]
    print("[case]", case, flush=True)
    net = dpsnn.dpsnn_build(W.swa(rate_bins_cap=64, **over), 1)
    assert net.stats()["schedule"] == want
    dpsnn.dpsnn_step(net, 3)
    assert dpsnn.dpsnn_sync(net) == 0
    net.close()
