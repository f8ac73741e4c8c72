"""Closures on a device that refuses cooperative launches: matrices of
half-precision keys go back to integers and are closed launch by launch."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

SCRIPT = """
import ctypes, sys
import numpy as np
refuse = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import torch
import oracle
import paper_2505_12976_amd as sz
ctx = sz.Context(0)
for dtype, m, top in (
        (np.uint16, 129, 90), (np.uint16, 200, 63489), (np.uint16, 200, 65536), (np.uint16, 1100, 40000),
        (np.int32, 129, 90), (np.int32, 300, 1 << 30),
        (np.int32, 1100, 3000),      # few values: ranks
        (np.int32, 1030, 64000),     # more than the keys hold, as many as ranks hold
        (np.int32, 1100, 1 << 23),   # too many values to rank
        (np.int32, 1100, 1 << 30)):  # too large to rank
    rng = np.random.default_rng(m + top % 1000)
    for mode in (oracle.WINNING_VOTES, oracle.MARGIN):
        print(dtype.__name__, m, top, mode, flush=True)
        d = rng.integers(0, top, size=(m, m))
        y, x = np.triu_indices(m, 1)
        k = min(len(y), top - 1, 70000)  # distinct weights, up to the largest, at random places
        at = rng.permutation(len(y))[:k]
        d[y[at], x[at]], d[x[at], y[at]] = np.arange(top - k, top), 0
        np.fill_diagonal(d, 0)
        want = oracle.closure(oracle.weights(d, mode))
        np.fill_diagonal(want, 0)
        before = refuse.refused_launches()
        ctx.reset_timing()
        ctx.set_timing(True)
        p = ctx.closure(torch.from_numpy(d.astype(dtype)).cuda(), mode)
        torch.cuda.synchronize()
        ctx.set_timing(False)
        assert refuse.refused_launches() > before and ctx.kernel_time("fw_rest")[0] > 0
        assert ctx.device_error() == 0
        assert np.array_equal(p.cpu().numpy().astype(np.int64), want)
print("all closed")
"""


def test_closure(tmp_path):
    so = str(tmp_path / "librefuse.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "refuse_cooperative.c"), "-o", so], check=True, capture_output=True)
    r = subprocess.run([sys.executable, "-c", SCRIPT, so, ROOT], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.splitlines()[-1] == "all closed", r.stdout[-400:] + r.stderr[-2000:]
