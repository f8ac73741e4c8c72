"""Outputs in rows of any pitch from any element on: what lies before the
first row and between the rows stays as it was, for each way the counts and
the closure are made; and repeated ids in full rankings too many for one pass."""
import numpy as np
import pytest

import oracle

from tests.test_gpu_bucketed import takes_buckets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


class Padded:
    """An m x m output whose rows of pitch m + extra start at element `offset` of a buffer of 77s."""

    def __init__(self, m, dtype, offset, extra):
        import torch
        self.flat = torch.full((offset + m * (m + extra) + 8,), 77, dtype=torch.int32, device="cuda:0")
        self.flat = self.flat.to(torch.uint16) if dtype == "u16" else self.flat
        self.offset, self.m, self.extra = offset, m, extra
        self.rows = self.flat[offset:offset + m * (m + extra)].view(m, m + extra)
        self.out = self.rows[:, :m]

    def check(self, want):
        flat = self.flat.cpu().numpy().astype(np.int64)
        rows = flat[self.offset:-8].reshape(self.m, self.m + self.extra)
        assert np.array_equal(rows[:, :self.m], want)
        assert (flat[:self.offset] == 77).all() and (flat[-8:] == 77).all() and (rows[:, self.m:] == 77).all()


PLACES = [(0, 0), (1, 0), (3, 2), (5, 1), (0, 7), (8, 8), (2, 13)]


def profile(way, rng):
    """(m, ballots) that are counted that way."""
    if way == "one pass":  # a share of the voters per workgroup, then a reduction
        m, n, L = 261, 3000, 261
    elif way == "one pass whole":  # all voters of a tile in one workgroup
        m, n, L = 261, 90, 30
    elif way == "one tile":
        m, n, L = 61, 200, 61
    elif way == "full":
        m, n, L = 4101, 40, 4101
    else:  # "bucketed", "atomic", and "dense": the same few ids on all ballots
        m, n, L = 4101, 20000 if way == "dense" else 200, 40
    b = np.argsort(rng.random((n, 60 if way == "dense" else m)), axis=1)[:, :L].astype(np.int32)
    if way != "full":
        b[1::2, L // 2:] = -1
    return m, b


@pytest.mark.parametrize("way", ["one pass", "one pass whole", "one tile", "full", "dense", "bucketed", "atomic"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("dtype", ["u16", "i32"])
def test_counts(ctx, way, weighted, dtype):
    import torch
    rng = np.random.default_rng(len(way))
    m, b = profile(way, rng)
    w = rng.integers(0, 4, size=len(b)).astype(np.uint32) if weighted else None
    want = oracle.pairwise(b, m, w)
    x = torch.from_numpy(b).cuda()
    xw = None if w is None else torch.from_numpy(w).cuda()
    ctx.set_sparse_count("atomic" if way == "atomic" else "bucketed")
    try:
        for offset, extra in PLACES:
            o = Padded(m, dtype, offset, extra)
            ctx.reset_timing()
            ctx.set_timing(True)
            ctx.pairwise(x, m, voter_weight=xw, dtype=dtype, out=o.out)
            torch.cuda.synchronize()
            ctx.set_timing(False)
            # (the sum of the weights counts as one launch of the decision)
            assert ctx.kernel_time("route")[0] == (0 if way.startswith("one") else 1) + weighted
            if way in ("dense", "bucketed") and not weighted:
                assert takes_buckets(b, m, False) == (way == "bucketed")
            assert ctx.device_error() == 0
            o.check(want)
    finally:
        ctx.set_sparse_count("bucketed")


@pytest.mark.parametrize("dtype", ["u16", "i32"])
@pytest.mark.parametrize("m", [7, 33, 61, 97, 128, 129, 261, 1101, 2053])  # (from 1024 on: value ranks for i32)
@pytest.mark.parametrize("schedule", ["auto", "phased"])
def test_closure(ctx, m, schedule, dtype):
    import torch
    rng = np.random.default_rng(m)
    d_np = rng.integers(0, 3000, size=(m, m))
    np.fill_diagonal(d_np, 0)
    want = oracle.closure(oracle.weights(d_np, oracle.WINNING_VOTES))
    np.fill_diagonal(want, 0)
    d = torch.from_numpy(d_np.astype(np.uint16 if dtype == "u16" else np.int32)).cuda()
    ctx.set_closure_schedule(schedule)
    try:
        for offset, extra in PLACES:
            o = Padded(m, dtype, offset, extra)
            ctx.closure(d, "winning_votes", out=o.out)
            torch.cuda.synchronize()
            assert ctx.device_error() == 0
            o.check(want)
    finally:
        ctx.set_closure_schedule("auto")


@pytest.mark.parametrize("ids", ["u16", "i32"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("m,n,L,row", [(4101, 40, 4101, 39), (4101, 40, 4100, 3), (4160, 300, 4160, 255)])
def test_repeated_id_of_a_full_ranking(ctx, m, n, L, row, weighted, ids):
    import torch
    import paper_2505_12976_amd as sz
    rng = np.random.default_rng(n)
    b = np.argsort(rng.random((n, m)), axis=1)[:, :L].astype(np.int32 if ids == "i32" else np.uint16)
    w = torch.ones(n, dtype=torch.int32, device="cuda").view(torch.uint32) if weighted else None
    good = b[row, 4000]
    for value, want in ((b[row, 17], sz.EBALLOT), (good, 0)):
        b[row, 4000] = value
        ctx.reset_timing()
        ctx.set_timing(True)
        d = ctx.pairwise(torch.from_numpy(b).cuda(), m, voter_weight=w, dtype="i32")
        torch.cuda.synchronize()
        ctx.set_timing(False)
        assert ctx.kernel_time("route")[0] == 1 + weighted and ctx.kernel_time("count_dense")[0] >= 1
        assert ctx.device_error() == want
    assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b.astype(np.int32), m))
