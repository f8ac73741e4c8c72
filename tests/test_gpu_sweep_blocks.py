"""Widest paths of one candidate on matrices of whole and partial column blocks
of 1024, with rows of whole 16-byte vectors and without: sweeps over written
weights and the check straight from the counts."""
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


@pytest.mark.parametrize("dtype", [np.uint16, np.int32])
@pytest.mark.parametrize("mode", [oracle.WINNING_VOTES, oracle.MARGIN])
@pytest.mark.parametrize("m,top", [(1020, 3000), (1024, 40), (1028, 3000), (1032, 40), (1030, 3000), (2048, 3000),
                                   (2056, 40), (2055, 3000)])
def test_blocks(ctx, m, top, mode, dtype):
    import torch
    rng = np.random.default_rng(m + top)
    d_np = rng.integers(0, top, size=(m, m))
    d_np[: m // 8] += top // 2  # (some that hardly anyone beats: small frontiers next to full ones)
    np.fill_diagonal(d_np, 0)
    w_np = oracle.weights(d_np.astype(np.int64), mode)
    p = oracle.closure(w_np)
    np.fill_diagonal(p, 0)
    d = torch.from_numpy(d_np.astype(dtype)).cuda()
    w, wt = ctx.weights(d, mode)
    for cand in (0, m // 8, m - 1):
        for verdict, p_from, p_to, _ in (ctx.verify_counts(d, cand, mode), ctx.verify(w, wt, cand)):
            assert np.array_equal(p_from.cpu().numpy().astype(np.int64), p[cand])
            assert np.array_equal(p_to.cpu().numpy().astype(np.int64), p[:, cand])
            assert int(verdict[1]) == (p[:, cand] > p[cand]).sum()
        got = ctx.widest_from(w, cand)
        assert np.array_equal(got.cpu().numpy().astype(np.int64), p[cand])
    torch.cuda.synchronize()
    assert ctx.device_error() == 0
