"""Matrices that start at any element and have any pitch: every pass over the
counts reads 16 bytes at a time whatever the alignment, with the last columns
and rows at the edges of its tiles, blocks and vectors."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 32, 33, 48, 49, 63, 64, 65, 96, 97, 128, 129, 131, 259, 1023, 1025, 1027, 1033]


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


def counts(m, seed, dtype):
    rng = np.random.default_rng(seed)
    d = rng.integers(0, 60 if m % 2 else 3000, size=(m, m))
    np.fill_diagonal(d, 0)
    return d.astype(dtype)


def view(d, offset, extra):
    """d on the GPU as rows of pitch m + extra that start at element `offset`."""
    import torch
    m = d.shape[0]
    flat = torch.full((offset + m * (m + extra),), 77, dtype=torch.int32, device="cuda:0")
    flat = flat.to(torch.uint16) if d.dtype == np.uint16 else flat
    v = flat[offset:].view(m, m + extra)[:, :m]
    v.copy_(torch.from_numpy(d).to("cuda:0"))
    return v


@pytest.mark.parametrize("dtype", [np.uint16, np.int32])
@pytest.mark.parametrize("offset,extra", [(0, 0), (1, 0), (3, 2), (5, 1), (0, 7)])
def test_any_alignment(ctx, dtype, offset, extra):
    import torch
    for m in SIZES:
        d_np = counts(m, 100 * m + offset, dtype)
        d = view(d_np, offset, extra)
        w_np = oracle.weights(d_np.astype(np.int64), oracle.WINNING_VOTES)
        p_np = oracle.closure(w_np)
        np.fill_diagonal(p_np, 0)
        out = view(np.zeros((m, m), dtype), offset, extra)
        p = ctx.closure(d, "winning_votes", out=out)
        assert np.array_equal(p.cpu().numpy().astype(np.int64), p_np), m
        bb = (p_np.T > p_np).sum(axis=1)
        is_winner, _ = ctx.winners(p)
        assert np.array_equal(is_winner.cpu().numpy() != 0, bb == 0), m
        order, beaten = ctx.ranking(p)
        assert np.array_equal(beaten.cpu().numpy(), bb), m
        f_np = oracle.features(d_np.astype(np.int64), 100.0, oracle.WINNING_VOTES)
        assert np.allclose(ctx.features(d, 100.0).cpu().numpy(), f_np, rtol=1e-5, atol=1e-6), m
        won, _, _ = ctx.winners_propagate(d)
        assert np.array_equal(won.cpu().numpy() != 0, bb == 0), m
        for cand in sorted({0, m // 2, m - 1}):
            verdict, p_from, p_to, _ = ctx.verify_counts(d, cand)
            assert np.array_equal(p_from.cpu().numpy().astype(np.int64), p_np[cand]), (m, cand)
            assert np.array_equal(p_to.cpu().numpy().astype(np.int64), p_np[:, cand]), (m, cand)
            assert int(verdict[1]) == bb[cand], (m, cand)
        w = view(w_np.astype(dtype), offset, extra)
        got = ctx.widest_from(w, m - 1)
        assert np.array_equal(got.cpu().numpy().astype(np.int64), p_np[m - 1]), m
    torch.cuda.synchronize()
    assert ctx.device_error() == 0
