"""The first slow-wave analysis of a process while another stream is being
captured in a graph (relaxed mode): the tables it uploads go on the call's own
stream, so that neither the call nor the capture fails."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes as C, sys
import torch
from paper_1902_08410_amd import dpsnn as D
g = torch.Generator(device="cuda").manual_seed(3)
c = torch.randint(0, 40, (200, 16, 2), dtype=torch.int32, device="cuda", generator=g)
a = torch.arange(1000.0, device="cuda")
side, own, L = torch.cuda.Stream(), torch.cuda.Stream(), D.lib()
torch.cuda.synchronize()


def analyse():
    wp, res = D._wave_params(0, 0, 0.5, 1, 2, 2, 1), D.DpsnnWaveResult()
    rc = getattr(L, sys.argv[1])(C.c_void_p(c.data_ptr()), 200, 4, 4, 2, 50, 0.1, 0, C.byref(wp),
                                 C.c_void_p(own.cuda_stream), C.byref(res), None, None, None, 0,
                                 None, None, None, 0)
    assert rc == 0, rc
    return res.n_transitions, res.n_waves


graph = torch.cuda.CUDAGraph()
with torch.cuda.stream(side):
    graph.capture_begin(capture_error_mode="relaxed")
    b = a * 2.0
    first = analyse()
    graph.capture_end()
assert first == analyse() and first[0] > 20
for k in range(3):
    a.add_(1.0)
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(b, a * 2.0)
print("done", first)
"""


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["dpsnn_waves_counts_static", "dpsnn_waves_counts"])
def test_first_analysis_beside_a_capture(entry):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case]", entry, flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD, entry], cwd=ROOT, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0 and "done" in r.stdout, r.stdout + r.stderr
