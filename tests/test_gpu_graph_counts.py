"""Counts captured in a HIP graph after one larger eager call, which sizes the
workspace: the smaller call takes other kernels than the larger one.  Every
replay is checked against the oracle, with new ballots in the captured buffer
and eager work and synchronisations between replays."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def ballots(rng, n, L, m):
    b = np.argsort(rng.random((n, m)), axis=1)[:, :L].astype(np.int32)
    b[np.arange(L)[None, :] >= rng.integers(0, L + 1, size=n)[:, None]] = -1
    return b


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("large,small", [
    ((4300, 3000, 9), (300, 2000, 7)),     # short ballots: routed, then in one pass
    ((4300, 3000, 9), (4200, 900, 9)),     # routed twice
    ((700, 900, 700), (70, 500, 70)),      # in one pass twice, whole tiles and then ranges
    ((4096, 70, 4096), (500, 64, 500)),
])
def test_smaller_count_in_a_graph(large, small, weighted):
    import torch
    import paper_2505_12976_amd as sz
    rng = np.random.default_rng(large[0] + small[0])
    ctx = sz.Context(0)
    try:
        def inputs(size):
            m, n, L = size
            b, w = ballots(rng, n, L, m), rng.integers(0, 50, size=n).astype(np.uint32)
            return b, w if weighted else None

        def gpu(b, w):
            return torch.from_numpy(b).cuda(), None if w is None else torch.from_numpy(w).cuda()

        m0, m = large[0], small[0]
        b0, w0 = inputs(large)
        tb0, tw0 = gpu(b0, w0)
        d0 = ctx.pairwise(tb0, m0, voter_weight=tw0)
        want0 = oracle.pairwise(b0, m0, w0)
        b, w = inputs(small)
        tb, tw = gpu(b, w)
        d = torch.empty((m, m), dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        assert np.array_equal(d0.cpu().numpy().astype(np.int64), want0)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            ctx.pairwise(tb, m, voter_weight=tw, out=d)
        for _ in range(3):
            d.fill_(-1)
            g.replay()
            torch.cuda.synchronize()
            assert ctx.device_error() == 0
            assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b, m, w))
            d0 = ctx.pairwise(tb0, m0, voter_weight=tw0)  # eager work on the same workspace
            b, w = inputs(small)
            tb.copy_(torch.from_numpy(b))
            if weighted:
                tw.copy_(torch.from_numpy(w))
            torch.cuda.synchronize()
            assert np.array_equal(d0.cpu().numpy().astype(np.int64), want0)
        del g
    finally:
        ctx.close()
