"""Rows with few synapses per delay: pieces of at most 8 synapses, whose
synapses share a wavefront's rows of lanes, against the oracle.

The cases sit at the edges: segments of 7, 8, 9 and 17 synapses, empty ones, a
wavefront's 64 pieces of 8 just filled, both sides of the line between short
and long pieces (20 synapses per delay), every entry format, lists and inboxes
that overflow, more target tiles than table entries, and plasticity.
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


def _tiny(**over):
    return W.tiny(**dict(dict(w=2, h=2, K=600, nu_ext_hz=[3500.0, 3500.0]), **over))


_AT2 = dict(d_min=2, d_max=2)
_HARD = dict(w=2, h=1, K=300, tau_arp=[0.0, 0.0], nu_ext_hz=[60000.0, 60000.0],
             J_mean=[0.2, -0.2], J_sd=[0.05, 0.05])
CASES = {
    "segment_7": _tiny(K_out=7, **_AT2),
    "segment_8_f16": _tiny(K_out=8, weight_dtype="f16", **_AT2),
    "segment_9_i8": _tiny(K_out=9, weight_dtype="i8", **_AT2),
    "segment_17_wide64": _tiny(K_out=17, acc_bits=64, q_frac_bits=32, **_AT2),
    # the fused schedule's own delivery of the first delay: 15 to 17 synapses, four
    # spikes at a time, many spikes a tile and few
    "segment_15_d1": _tiny(K_out=15, d_min=1, d_max=1),
    "segment_16_d1_f16": _tiny(K_out=16, weight_dtype="f16", d_min=1, d_max=1),
    "segment_17_d1_i8": _tiny(K_out=17, weight_dtype="i8", d_min=1, d_max=1),
    "bursts_16_d1": W.tiny(K_out=16, d_min=1, d_max=1, **_HARD),
    "few_spikes_d1": _tiny(K_out=18, d_min=1, d_max=1, nu_ext_hz=[1500.0, 1500.0]),
    "inbox_full_d1": _tiny(K_out=18, queue_cap=3, d_min=1, d_max=1),
    "segment_20_d1": _tiny(K_out=20, d_min=1, d_max=1),
    "segment_21_d1": _tiny(K_out=21, d_min=1, d_max=1),
    "line_short": _tiny(K_out=100, d_max=5), "line_long": _tiny(K_out=101, d_max=5),
    "delays_64_i8_q32": _tiny(K_out=200, d_max=64, weight_dtype="i8", acc_bits=64, q_frac_bits=32),
    "wide32": _tiny(K_out=30, J_mean=[35.0, -40.0], J_sd=[5.0, 5.0]),
    # most neurons fire in a step: full wavefronts of 64 pieces of 8 synapses
    "bursts_8": W.tiny(K_out=8, **_AT2, **_HARD),
    "bursts_16_f16": W.tiny(K_out=16, weight_dtype="f16", **_AT2, **_HARD),
    "lists_full": W.tiny(K_out=16, queue_cap=2, d_min=1, d_max=2, **_HARD),
    "lists_full_i8": W.tiny(K_out=16, queue_cap=2, weight_dtype="i8", **_AT2, **_HARD),
    "inbox_full": _tiny(K_out=60, queue_cap=3),
    # long pieces over several parts of the lists and a tile just begun
    "parts_long": W.tiny(w=17, h=1, K=1025, K_out=130, nu_ext_hz=[2600.0, 2600.0]),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_short_rows_bit_exact(L, case):
    print("[case]", case, flush=True)
    sys.stdout.flush()
    p = dict(CASES[case], spike_log_cap=1 << 21, rate_bins_cap=256)
    steps = 30 if p["tau_arp"][0] == 0.0 else 200
    for order in ((1, 0, 2), (0, 2, 1)):
        net, orc = L.dpsnn_build(p, 6), O.Oracle(p, 6, store_rows=True)
        for sched in order:
            L.dpsnn_set_schedule(net, sched)
            L.dpsnn_step(net, steps)
        orc.step(steps * len(order))
        assert _compare(L, net, orc, (case, order)) > 20
        net.close()


@pytest.mark.parametrize("K_out,steps,over", [
    (16, 5, dict(tau_arp=[0.0, 0.0], nu_ext_hz=[60000.0, 60000.0])),
    (512, 6, dict(nu_ext_hz=[300.0, 300.0]))])
def test_more_target_tiles_than_table_entries_at_delay_2(L, K_out, steps, over):
    """46x46 modules (2583 tiles), every synapse remote and its module drawn
    almost uniformly, one delay of two steps, so that every schedule delivers
    through its table (2048 entries; 1024 of the persistent schedule).  With
    16 synapses all neurons fire in every step and full slices of short pieces
    bring 4096 events (2048 of the persistent schedule), with 512 the last
    steps bring full slices of long ones: about 2050 (1400) distinct tiles and
    more, so runs make reservations of their own."""
    p = W.grid(46, 46, "swa", K_out=K_out, frac_local=[0.0, 0.0], spike_log_cap=1 << 24,
               rate_bins_cap=64, **over, **_AT2, **{"lambda": 100.0})
    print("[case] tables full", K_out, flush=True)
    orc = O.Oracle(p, 8, store_rows=False)
    orc.step(steps)
    for sched in (0, 1, 2):
        print("[case] schedule", sched, flush=True)
        net = L.dpsnn_build(p, 8)
        L.dpsnn_set_schedule(net, sched)
        L.dpsnn_step(net, steps)
        assert _compare(L, net, orc, (sched, K_out)) > 100000
        net.close()
    orc.close()


def test_plastic_short_rows(L):
    p = _tiny(K_out=24, d_max=5, spike_log_cap=1 << 20, rate_bins_cap=64,
              **W.stdp(stdp_update_steps=70, stdp_eta=5.0))
    print("[case] plastic short rows", flush=True)
    net, orc = L.dpsnn_build(p, 4), O.Oracle(p, 4, store_rows=True)
    L.dpsnn_step(net, 300)
    orc.step(300)
    assert _compare(L, net, orc, "plastic") > 100
    net.close()


def test_short_rows_are_not_dear(L):
    """48x48 modules: 100 synapses a neuron at 96 Hz make half the events of 1000
    at 18 Hz.  Their delivery took 3 times as long when each segment had 64
    lanes of its own, and the update twice as long for an atomic per segment."""
    ms = {}
    for K_out in (100, 1000):
        k = 1000 / K_out
        p = W.grid(48, 48, "swa", K_out=K_out, J_mean=[0.5 * k, -2.0 * k],
                   J_sd=[0.1 * k, 0.4 * k], rate_bins_cap=64)
        print("[case] time", K_out, flush=True)
        net = L.dpsnn_build(p, 5)
        L.dpsnn_set_schedule(net, 1)
        L.dpsnn_step(net, 300)
        ms[K_out] = L.dpsnn_profile_steps(net, 200)
        net.close()
    print(ms, flush=True)
    assert ms[100][0] < 1.8 * ms[1000][0] and ms[100][1] < 2.0 * ms[1000][1]
