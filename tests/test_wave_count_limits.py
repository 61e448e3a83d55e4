"""Counts at and past the wave analysis's table of logarithms (65537 entries,
log(0) .. log(65536), for counts up to 65535): the decision that keeps the
kernels inside the table, on the CPU, and the entry points on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HELP = os.path.join(ROOT, "tests", "helpers")


def test_table_guard_does_not_wrap(tmp_path):
    """Entries up to mx + 1 are read, in 64 bits: the table serves mx exactly
    if mx + 2 <= lnt_n, also where mx + 2 passes 32 bits."""
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are missing")
    exe = str(tmp_path / "guard")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1902_08410_amd", "csrc"), "-o", exe,
                    os.path.join(HELP, "wave_table_guard.cpp")], check=True, capture_output=True)
    cases = [(n, mx) for n in (2, 65537, 70002, 2**32 - 1)
             for mx in (0, 1, 65535, 65536, 70000, 70001, 2**31, 2**32 - 4, 2**32 - 3,
                        2**32 - 2, 2**32 - 1)]
    out = subprocess.run([exe], input="".join("%d %d\n" % c for c in cases), text=True,
                         capture_output=True, check=True).stdout.split()
    assert [int(x) for x in out] == [int(mx + 2 <= n) for n, mx in cases]


def _counts(top):
    """One module of two counts `top` between quiet bins, three of plain Up states."""
    rng = np.random.default_rng(3)
    c = rng.poisson(1.5, size=(200, 4, 2)).astype(np.uint32)
    for k0 in range(20, 180, 40):
        c[k0:k0 + 15, :, 0] += np.uint32(30)
    c[60:62, 2, 1] = 0
    c[60:62, 2, 0] = top
    return c


@pytest.mark.gpu
@pytest.mark.parametrize("top", [65535, 65536, 70000])
def test_counts_around_the_table(top):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_08410_amd import dpsnn
    c = _counts(top)
    kw = dict(noise_var=0.25, seed=5, min_down=2, min_up=2, min_modules=1)
    print("[case] counts up to", top, flush=True)
    ref = O.waves(c, 2, 2, 50, 0.1, **kw)
    t = torch.from_numpy(c.view(np.int32)).cuda()
    calls = [dpsnn.dpsnn_waves_counts]
    if top <= 65535:
        calls.append(dpsnn.dpsnn_waves_counts_static)
    else:
        with pytest.raises(dpsnn.DpsnnError) as e:
            dpsnn.dpsnn_waves_counts_static(t, 2, 2, 50, 0.1, **kw)
        assert e.value.code == -8
    for f in calls:
        got = f(t, 2, 2, 50, 0.1, **kw)
        assert got["n_transitions"] == len(ref["T"]) > 8
        for k in ("module", "T", "wave", "n", "t0"):
            assert np.array_equal(got[k], ref[k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("top", [2**32 - 2, 2**32 - 1])
def test_counts_past_32_bit_tables_are_refused(top):
    """-2 and -1 of an int32 tensor: an error from both entries, and the next
    analysis is unharmed."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_08410_amd import dpsnn
    kw = dict(noise_var=0.25, seed=5, min_down=2, min_up=2, min_modules=1)
    print("[case] counts up to", top, flush=True)
    t = torch.from_numpy(_counts(top).view(np.int32)).cuda()
    for f, code in ((dpsnn.dpsnn_waves_counts_static, -8), (dpsnn.dpsnn_waves_counts, -2)):
        with pytest.raises(dpsnn.DpsnnError) as e:
            f(t, 2, 2, 50, 0.1, **kw)
        assert e.value.code == code
    c = _counts(40)
    ref = O.waves(c, 2, 2, 50, 0.1, **kw)
    got = dpsnn.dpsnn_waves_counts(torch.from_numpy(c.view(np.int32)).cuda(), 2, 2, 50, 0.1, **kw)
    assert np.array_equal(got["T"], ref["T"])
