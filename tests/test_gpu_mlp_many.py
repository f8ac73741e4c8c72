"""The loss over many elections: on both sides of the number that gets a
workgroup each (four per CU), against the float64 loss, and over more
elections than workgroups of 256 threads fit one launch."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


def t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("over", [-1, 0, 1, 3075])
def test_loss_around_the_rule(ctx, over):
    import torch
    E = 4 * torch.cuda.get_device_properties(0).multi_processor_count + over
    rng = np.random.default_rng(5)
    sizes = rng.integers(0, 71, size=E)
    sizes[[0, E // 2, E - 1]] = 1, 300, 64
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    M = int(off[-1])
    score = rng.standard_normal(M).astype(np.float32)
    win = (rng.random(M) < 0.1).astype(np.uint8)
    ds, loss = ctx.mlp_loss(t(score), t(off), t(win))
    ds, loss = ds.cpu().numpy(), loss.cpu().numpy()
    s64 = score.astype(np.float64)
    for e in range(E):
        a, b = off[e], off[e + 1]
        want, want_ds = omlp.seg_loss(s64[a:b], np.array([0, b - a]), win[a:b], np.float64) if b > a else (0.0, 0.0)
        # sums of at most five values per lane and six steps over the lanes, each within 2^-24, and two logarithms
        assert abs(loss[e] - want) <= 1e-5, e
        assert np.all(np.abs(ds[a:b] * E - want_ds) <= 1e-5), e
    # both kernels add in the same order: the first elections' losses do not depend on how many follow
    head = E // 2
    _, few = ctx.mlp_loss(t(score[:off[head]]), t(off[:head + 1]), t(win[:off[head]]))
    assert np.array_equal(few.cpu().numpy(), loss[:head])


def test_more_elections_than_workgroups_fit_a_launch(ctx):
    E = (1 << 24) + 5
    off = np.arange(E + 1, dtype=np.int64)
    off[-1] += 2  # the last election has three rows, every other one
    M = int(off[-1])
    score = np.zeros(M, dtype=np.float32)
    score[-3:] = 0.5, -1.0, 2.0
    win = np.zeros(M, dtype=np.uint8)
    win[-2] = 1
    ds, loss = ctx.mlp_loss(t(score), t(off), t(win))
    want, want_ds = omlp.seg_loss(score[-3:].astype(np.float64), np.array([0, 3]), win[-3:], np.float64)
    loss = loss.cpu().numpy()
    assert np.all(loss[:-1] == 0) and abs(loss[-1] - want) <= 1e-5
    ds = ds.cpu().numpy()
    assert np.all(ds[:-3] == 0) and np.all(np.abs(ds[-3:] * E - want_ds) <= 1e-5)
