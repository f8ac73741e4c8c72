"""Voter weights of every width: bit planes up to 8 bits, digits of four bits
beyond, sixteen bits at a time, in the one-pass count and in the routed count
of full rankings, with single heavy voters among light ones."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("m,n,L", [(37, 65, 37), (130, 33, 20), (64, 1, 64), (300, 700, 300), (4200, 40, 4200)])
@pytest.mark.parametrize("bits", [1, 4, 7, 8, 9, 12, 13, 16, 17, 20, 24, 25, 31, 32])
def test_weight_bits(ctx, m, n, L, bits):
    import torch
    rng = np.random.default_rng(100 * bits + m)
    b = np.argsort(rng.random((n, m)), axis=1)[:, :L].astype(np.int32)
    b[::3, L // 2:] = -1
    w = rng.integers(0, 1 << min(bits, 4), size=n, dtype=np.int64)
    top = (1 << bits) - 1
    w[n // 2] = top if bits < 31 else (1 << 31) - 1 - 16 * n  # (every count below 2^31)
    if bits == 32:  # the top bit of a weight; its voter prefers nobody
        w[n // 2], b[n // 2] = 1 << 31, -1
    elif bits < 31:
        light = (1 << 31) // (2 * n)
        w[:n // 3] = rng.integers(0, min(top + 1, light), size=n // 3)
    w = w.astype(np.uint32)
    d = ctx.pairwise(torch.from_numpy(b).cuda(), m, voter_weight=torch.from_numpy(w).cuda(), dtype="i32")
    torch.cuda.synchronize()
    want = oracle.pairwise(b, m, w)
    assert want.max() < 1 << 31
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), want)
