"""Batch finish on 16-bit values: half-precision keys up to their largest
value and integers above it, every closure schedule, block edges."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 16, 17, 31, 33, 48, 49, 63, 64, 65, 96, 97, 128, 129, 192, 193, 257]


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


def tournament(m, top, seed):
    """Counts d[x][y] up to top (both top and 1 among the winning ones)."""
    rng = np.random.default_rng(seed)
    d = rng.integers(0, top + 1, size=(m, m))
    d[rng.random((m, m)) < 0.4] = 0
    if m > 2:
        d[0, 1], d[1, 0], d[1, 2], d[2, 1] = top, 0, 1, 0
    np.fill_diagonal(d, 0)
    return d


@pytest.mark.parametrize("schedule", ["auto", "tiled32", "tiled64", "tiled128"])
@pytest.mark.parametrize("top", [1, 63488, 63489, 65535])
def test_batch_finish_value_ranges(ctx, schedule, top):
    import torch
    from paper_2505_12976_amd.batch import Packed, alloc_outputs
    ds = [tournament(m, top, 10 * m + top) for m in SIZES]
    els, mat, vec = [], 0, 0
    for m in SIZES:
        els.append((0, top, m, m, mat, vec))
        mat += m * m
        vec += m
    ctx.batch_set_closure(16, 1, 576, schedule)
    plan = ctx.batch_plan(els, "u16", "winning_votes", closure_only=True)
    ctx.batch_set_closure(16, 1, 576, "auto")
    outs = alloc_outputs(Packed(None, els, mat, vec), torch.device("cuda", 0))
    outs["d"].copy_(torch.from_numpy(np.concatenate([d.reshape(-1) for d in ds]).astype(np.int32)))
    ctx.batch_run(plan, None, outs["d"], outs["is_winner"], p=outs["p"], n_winners=outs["n_winners"],
                  beaten_by=outs["beaten_by"], order=outs["order"])
    torch.cuda.synchronize()
    assert ctx.device_error() == 0
    p_all, bb_all = outs["p"].cpu().numpy(), outs["beaten_by"].cpu().numpy()
    for (_, _, m, _, mo, vo), d in zip(els, ds):
        p = oracle.closure(oracle.weights(d.astype(np.int64), oracle.WINNING_VOTES))
        np.fill_diagonal(p, 0)
        assert np.array_equal(p_all[mo:mo + m * m].reshape(m, m), p), (schedule, top, m)
        bb = (p.T > p).sum(axis=1)
        assert np.array_equal(bb_all[vo:vo + m], bb), (schedule, top, m)
        assert np.array_equal(outs["is_winner"].cpu().numpy()[vo:vo + m] != 0, bb == 0), (schedule, top, m)
    plan.destroy()
