"""The autotuner: the spike-list kinds launch the same kernels, so it leaves the
caller's kind as it is; the number of steps it takes does not depend on that."""
import pytest

import oracle as O
from paper_1902_08410_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_list_kind_stays_as_set():
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_08410_amd import dpsnn as L
    p = W.tiny(w=3, h=3, K=400, K_out=120, nu_ext_hz=[3000.0, 3000.0], spike_log_cap=1 << 20,
               rate_bins_cap=1024)
    print("[case] autotune", flush=True)
    net, orc = L.dpsnn_build(p, 9), O.Oracle(p, 9, store_rows=True)
    for kind in (0, 1, 2, 0, 1, 2):
        L.dpsnn_set_delivery(net, 0, kind)
        t0 = net.stats()["t"]
        L.dpsnn_autotune(net, 20)
        st = net.stats()
        # fused, persistent and 4 grids of each kind; two runs of 20 steps each
        assert st["spike_lists"] == kind and st["t"] - t0 == 2 * 20 * (2 + 3 * 4)
        orc.step(st["t"] - t0)
    # a grid asked for by the number that is reported for the library's own
    L.dpsnn_set_schedule(net, 1)
    L.dpsnn_set_delivery(net, 256)
    L.dpsnn_step(net, 100)
    orc.step(100)
    assert net.stats()["deliver_blocks"] == 256
    assert np.array_equal(L.dpsnn_read_slots(net), orc.ring())
    net.close()
