"""The lists of pieces that wait for their step: their room and what happens
past it, against the oracle.

The room follows queue_cap: lists of a few pieces per tile overflow at once,
pieces that no longer fit are added into the slots by whole wavefronts, in
every entry format and schedule.  With the default, bursts of a network with a
single delay (16 pieces a spike) fit, and the update does not pay for them.
"""
import sys

import numpy as np
import pytest

import oracle as O
from paper_1902_08410_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_08410_amd import dpsnn
    dpsnn.lib()
    return dpsnn


def _compare(L, net, orc, what):
    st, ids = L.dpsnn_read_spikes(net)
    ost, oids = orc.spikes()
    assert np.array_equal(st, ost) and np.array_equal(ids, oids), what
    V, c, r = L.dpsnn_read_state(net)
    oV, oc, orr = orc.state()
    assert np.array_equal(V.astype(np.float64), oV), what
    assert np.array_equal(c.astype(np.float64), oc), what
    assert np.array_equal(r.astype(np.int32), orr), what
    assert np.array_equal(L.dpsnn_read_slots(net), orc.ring()), what
    return len(st)


# most neurons fire in a step; rows of 200 synapses over one or two delays
_HARD = dict(w=2, h=1, K=300, K_out=200, tau_arp=[0.0, 0.0], nu_ext_hz=[60000.0, 60000.0],
             J_mean=[0.2, -0.2], J_sd=[0.05, 0.05])
FORMATS = {
    "packed": dict(d_min=1, d_max=1),
    "packed_2": dict(d_min=2, d_max=3),
    "wide64": dict(d_min=2, d_max=2, acc_bits=64, q_frac_bits=32),
    "wide32": dict(d_min=1, d_max=2, J_mean=[33.0, -33.0], J_sd=[0.5, 0.5]),
    "f16": dict(d_min=2, d_max=3, weight_dtype="f16"),
    "i8": dict(d_min=1, d_max=1, weight_dtype="i8", acc_bits=64, q_frac_bits=32),
}


@pytest.mark.parametrize("cap", [2, 40])
@pytest.mark.parametrize("fmt", sorted(FORMATS))
def test_pieces_past_the_end_of_a_list(L, fmt, cap):
    p = W.tiny(**dict(_HARD, queue_cap=cap, spike_log_cap=1 << 20, rate_bins_cap=64,
                      **FORMATS[fmt]))
    print("[case] list full", fmt, cap, flush=True)
    sys.stdout.flush()
    for order in ((1, 0), (0, 2, 1)):
        net, orc = L.dpsnn_build(p, 6), O.Oracle(p, 6, store_rows=True)
        for sched in order:
            L.dpsnn_set_schedule(net, sched)
            L.dpsnn_step(net, 12)
        orc.step(12 * len(order))
        assert _compare(L, net, orc, (fmt, cap, order)) > 500
        net.close()


@pytest.mark.parametrize("over", [
    dict(queue_cap=64, d_max=20), dict(queue_cap=64, d_min=64, d_max=127),
    dict(queue_cap=256, d_max=20, weight_dtype="f16"), dict(d_max=20),
    dict(d_max=1, K_out=1000), dict(d_min=20, d_max=20, K_out=1000)])
def test_lists_take_no_more_than_cap_entries_per_slot(L, over):
    """Inboxes (4 cap entries a tile) and lists within (D + 4) x cap entries a
    tile: what a caller sizes with queue_cap."""
    p = W.tiny(**dict(dict(w=16, h=1, K=1024, K_out=8, queue_cap=0), **over))
    print("[case]", over, flush=True)
    net = L.dpsnn_build(p, 1)
    s, D, tiles, N = net.stats(), p["d_max"] + 1, 16, 16 * 1024
    eb = 4 if p["weight_dtype"] == "f16" else 8
    counters = 64 * D + 2 * 64 * tiles + 4 * D * tiles
    extra = s["bytes_state"] - (9 + 4 * D) * N - counters
    assert 0 < extra <= tiles * (D + 4) * s["queue_cap"] * eb
    net.close()


def test_bursts_of_a_single_delay_fit_their_lists(L):
    """48x48 modules, one delay of one step: spikes come in bursts of a few per
    cent of the neurons, 16 pieces each.  Listing them is a small part of
    delivering them (the update took 4 times the delivery when they overflowed)."""
    p = W.grid(48, 48, "swa", d_min=1, d_max=1, rate_bins_cap=64)
    print("[case] bursts, one delay", flush=True)
    net = L.dpsnn_build(p, 5)
    L.dpsnn_set_schedule(net, 1)
    L.dpsnn_step(net, 300)
    upd, dlv = L.dpsnn_profile_steps(net, 200)
    print("update %.1f us, delivery %.1f us" % (upd * 5, dlv * 5), flush=True)
    net.close()
    assert upd < dlv
