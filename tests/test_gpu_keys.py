"""uint16 closures on half-precision keys: every 16-bit value, both tiles, and
matrices with values that have no key in order (closed as integers)."""
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


def counts(m, low, top, seed):
    """A tournament whose winning weights are spread over low .. top, both ends among them."""
    rng = np.random.default_rng(seed)
    w = rng.integers(low, top + 1, size=(m, m))
    w[0, 1], w[1, 2], w[2, 3] = top, low, (low + top) // 2
    wins = np.triu(rng.random((m, m)) < 0.5, 1)
    wins[0, 1] = wins[1, 2] = wins[2, 3] = True
    wins = wins | (np.tril(~wins.T, -1))
    d = np.where(wins, w, 0)
    d[rng.random((m, m)) < 0.3] = 0
    d[0, 1] = top
    np.fill_diagonal(d, 0)
    return d.astype(np.uint16)


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("low,top", [(0, 3), (31700, 31790), (1, 63488), (63000, 63489), (1, 65535), (63488, 63488)])
@pytest.mark.parametrize("m", [130, 257])
def test_u16_closure_every_value_range(ctx, tile, low, top, m):
    import torch
    d = counts(m, low, top, 7 * m + top + low)
    w = oracle.weights(d.astype(np.int64), oracle.WINNING_VOTES)
    want = oracle.closure(w)
    ctx.set_closure_tile(tile)
    try:
        got = {}
        for schedule in ("auto", "phased"):
            ctx.set_closure_schedule(schedule)
            p = ctx.closure(torch.from_numpy(d).cuda())
            torch.cuda.synchronize()
            got[schedule] = p.cpu().numpy().astype(np.int64)
    finally:
        ctx.set_closure_schedule("auto")
        ctx.set_closure_tile(0)
    assert ctx.device_error() == 0
    for schedule, p in got.items():
        assert np.array_equal(p, want), schedule
