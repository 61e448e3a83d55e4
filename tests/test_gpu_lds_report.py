"""stats.lds_bytes: the LDS of the larger kernel that the current schedule
launches, by entry size, slot width, rows and plasticity."""
import pytest

from paper_1902_08410_amd import workloads as W

pytestmark = pytest.mark.gpu


def _deliver(threads, pieces, bits, entry):
    """Prefix of 1024 parts, two tables, the slice's entries and their 2-byte
    keys, a word per wavefront and a flag."""
    n = 4096 + 8 * 2**bits + threads * pieces * (entry + 2) + threads // 16 + 4
    return -(-n // entry) * entry


def _update(slot):
    return 4096 + 1024 * slot + 16


WIDE = dict(acc_bits=64, q_frac_bits=32)
CASES = [  # split: pieces per wavefront; entry and slot bytes
    (dict(K_out=1000), 16, 4, 4), (dict(K_out=1000, weight_dtype="f16"), 16, 4, 4),
    (dict(K_out=1000, weight_dtype="i8", **WIDE), 16, 4, 8), (dict(K_out=1000, **WIDE), 8, 8, 8),
    (dict(K_out=100), 8, 4, 4), (dict(K_out=100, **WIDE), 8, 8, 8),
    (dict(K_out=1000, **W.stdp()), 8, 4, 4),
]


@pytest.mark.parametrize("over,pieces,entry,slot", CASES)
def test_lds_bytes_of_the_schedule(over, pieces, entry, slot):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_08410_amd import dpsnn as L
    print("[case]", over, flush=True)
    net = L.dpsnn_build(W.swa(rate_bins_cap=16, **over), 1)
    want = {1: max(_update(slot), _deliver(512, pieces, 11, entry)),
            0: max(2 * _update(slot), _deliver(512, 8, 11, entry)),
            2: max(_update(slot), _deliver(256, 8, 10, entry))}
    for sched in ((1,) if over.get("plastic") else (1, 0, 2)):
        L.dpsnn_set_schedule(net, sched)
        assert net.stats()["lds_bytes"] == want[sched], sched
    net.close()
