"""Handles without inboxes: every event is added into its slot when it is
emitted, 256 synapses of a row at a time.  Rows of one synapse less and one
more than that, in each format and schedule, against the oracle; and the time
of a small network's step."""
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


@pytest.mark.parametrize("K_out,over", [
    (1, dict()), (63, dict(weight_dtype="f16")), (255, dict(d_max=20)), (256, dict(d_min=2)),
    (257, dict(weight_dtype="i8", acc_bits=64, q_frac_bits=32)),
    (513, dict(acc_bits=64, q_frac_bits=32)), (300, dict(queue_cap=0, d_min=100, d_max=140))])
def test_rows_into_slots_bit_exact(L, K_out, over):
    p = W.tiny(**dict(dict(w=2, h=2, K=600, K_out=K_out, queue_cap=-1, spike_log_cap=1 << 20,
                           nu_ext_hz=[3500.0, 3500.0], rate_bins_cap=64), **over))
    print("[case]", K_out, over, flush=True)
    net, orc = L.dpsnn_build(p, 6), O.Oracle(p, 6, store_rows=True)
    assert net.stats()["queue_cap"] == 0
    for sched in (1, 0, 2):
        L.dpsnn_set_schedule(net, sched)
        L.dpsnn_step(net, 150)
    orc.step(450)
    st, ids = L.dpsnn_read_spikes(net)
    ost, oids = orc.spikes()
    assert len(st) > 100 and np.array_equal(st, ost) and np.array_equal(ids, oids)
    assert np.array_equal(L.dpsnn_read_slots(net), orc.ring())
    net.close()


def test_small_step_without_inboxes(L):
    """5000 neurons, 1000 synapses, 12 spikes a step: the rows' additions take
    about as long as the update (twice as long when each row's loads waited
    for one another)."""
    net = L.dpsnn_build(W.swa(queue_cap=-1, rate_bins_cap=64), 5)
    L.dpsnn_set_schedule(net, 1)
    L.dpsnn_step(net, 500)
    ms = [L.dpsnn_profile_steps(net, 200) for _ in range(3)]
    upd, dlv = sorted(ms, key=sum)[0]
    print("[case] update %.1f us, delivery %.1f us" % (upd * 5, dlv * 5), flush=True)
    net.close()
    assert dlv < 1.6 * upd
