"""Reading rows back: a few in one copy, many some at a time, the same bytes
either way; and what one row costs."""
import time

import numpy as np
import pytest

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
    (1, dict()), (63, dict(weight_dtype="i8")), (65, dict(weight_dtype="f16")), (1000, dict()),
    (1025, dict(K=1500, weight_dtype="i8")), (4096, dict(K=4200, weight_dtype="f16"))])
def test_rows_alone_and_in_bulk(L, K_out, over):
    p = W.swa(**dict(dict(grid_w=2, grid_h=1, K_out=K_out, rate_bins_cap=4), **over))
    print("[case]", K_out, over, flush=True)
    net = L.dpsnn_build(p, 11)
    n = min(1200, 2 * p["K"])
    tgt, w, dk = L.dpsnn_read_rows(net, 0, n)
    edge = (1 << 16) // K_out  # most rows that come back in one copy
    for first, count in [(0, 1), (7, 3), (n - 1, 1), (5, min(edge, n - 5)),
                         (3, min(edge + 1, n - 3))]:
        for got, all_ in zip(L.dpsnn_read_rows(net, first, count), (tgt, w, dk)):
            assert np.array_equal(got, all_[first:first + count]), (first, count)
    key = tgt.astype(np.int64) * 64 + dk
    assert (np.diff(key, axis=1) >= 0).all()
    # targets alone, delays alone, efficacies alone
    a, b, c = np.zeros_like(tgt[:2]), np.zeros_like(w[:2]), np.zeros_like(dk[:2])
    for ptrs in ((a, None, None), (None, b, None), (None, None, c)):
        assert L.lib().dpsnn_read_rows(net.h, 4, 2, *[L._ptr(x) for x in ptrs]) == 0
    assert np.array_equal(a, tgt[4:6]) and np.array_equal(b, w[4:6]) and np.array_equal(c, dk[4:6])
    net.close()


def test_one_row_is_cheap(L):
    """A row of 1000 synapses against the state of 5000 neurons (three copies):
    1.3 of its time (2.3 with one wavefront's sort and a copy for each part)."""
    net = L.dpsnn_build(W.swa(rate_bins_cap=4), 3)
    ts = {"row": [], "state": []}
    for _ in range(50):
        for k, f in (("row", lambda: L.dpsnn_read_rows(net, 5, 1)),
                     ("state", lambda: L.dpsnn_read_state(net))):
            t = time.perf_counter()
            f()
            ts[k].append(time.perf_counter() - t)
    us = {k: 1e6 * np.median(v) for k, v in ts.items()}
    print("[case] us", us, flush=True)
    net.close()
    assert us["row"] < 1.9 * us["state"]
