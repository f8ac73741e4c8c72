"""Bit-plane pairwise counts against the oracle at the edges of their groups
of 32 voters, tiles of 128 candidates and numbers of rank bits, with and
without voter weights, full rankings and truncated ballots mixed."""
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


def ballots(rng, n, m, L, cut, ids):
    b = np.argsort(rng.random((n, m)), axis=1)[:, :L].astype(np.int64)
    short = rng.random(n) < cut
    k = rng.integers(0, L + 1, size=n)
    b[short[:, None] & (np.arange(L)[None, :] >= k[:, None])] = -1
    return b.astype(np.int32) if ids == "i32" else b.astype(np.uint16)


@pytest.mark.parametrize("route", ["bucketed", "atomic"])  # atomic also takes small elections off the one-pass count
@pytest.mark.parametrize("ids", ["u16", "i32"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("m,n,L,cut", [
    (1, 5, 1, 0.5), (2, 33, 2, 0.5), (3, 32, 2, 0.0), (17, 31, 16, 0.3), (64, 65, 64, 0.0), (65, 1, 65, 0.0),
    (127, 97, 127, 0.4), (128, 64, 127, 0.4), (129, 600, 129, 0.2), (255, 40, 7, 0.5), (257, 2000, 256, 0.5),
    (1025, 70, 1025, 0.3), (2049, 33, 2049, 0.1), (1100, 3000, 9, 0.2), (700, 999, 699, 1.0),
    (5, 30000, 5, 0.3), (300, 20000, 300, 0.1), (4200, 3000, 9, 0.2), (1500, 2100, 700, 0.5)])
def test_counts(ctx, m, n, L, cut, weighted, ids, route):
    import torch
    rng = np.random.default_rng(m * 1000 + n)
    b = ballots(rng, n, m, L, cut, ids)
    w = rng.integers(0, 1 << 16 if m % 2 else 41, size=n).astype(np.uint32) if weighted else None
    ctx.set_sparse_count(route)
    try:
        d = ctx.pairwise(torch.from_numpy(b).cuda(), m, dtype="i32",
                         voter_weight=None if w is None else torch.from_numpy(w).cuda())
    finally:
        ctx.set_sparse_count("bucketed")
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b, m, w))


@pytest.mark.parametrize("m,L", [(40, 40), (40, 12), (1500, 1500)])
def test_repeated_id_is_an_error(ctx, m, L):
    import torch
    import paper_2505_12976_amd as sz
    b = ballots(np.random.default_rng(3), 50, m, L, 0.0, "u16")
    b[37, 5] = b[37, 2]
    ctx.pairwise(torch.from_numpy(b).cuda(), m)
    assert ctx.device_error() == sz.EBALLOT
    b[37, 5:] = 0xFFFF
    ctx.pairwise(torch.from_numpy(b).cuda(), m)
    assert ctx.device_error() == 0


@pytest.mark.parametrize("dtype", ["u16", "i32"])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 127, 128, 129])
def test_small_closure_and_ranking(ctx, m, mode, dtype):
    """One-workgroup closure, winners and ranking at the edges of their sizes."""
    import torch
    rng = np.random.default_rng(m + mode)
    b = ballots(rng, 37, m, m, 0.4, "u16")
    want = oracle.schulze(b, m, mode)
    d = torch.from_numpy(want["d"].astype(np.uint16 if dtype == "u16" else np.int32)).cuda()
    pad = torch.zeros((m, m + 3), dtype=d.dtype, device="cuda")[:, :m]  # a leading dimension above m
    p = ctx.closure(d, mode, out=pad)
    is_w, nw = ctx.winners(p)
    order, beaten = ctx.ranking(p)
    assert ctx.device_error() == 0
    assert np.array_equal(p.cpu().numpy().astype(np.int64), want["p"])
    assert np.array_equal(is_w.cpu().numpy().astype(bool), want["is_winner"])
    assert int(nw.cpu()[0]) == int(want["is_winner"].sum())
    assert np.array_equal(order.cpu().numpy(), want["order"])
    assert np.array_equal(beaten.cpu().numpy(), want["beaten_by"])


@pytest.mark.parametrize("route", ["bucketed", "atomic"])
@pytest.mark.parametrize("ids", ["u16", "i32"])
@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("m,n,L", [(70, 3, 70), (9, 1, 9), (300, 77, 299), (131, 40, 66), (2100, 5, 2100)])
def test_ballot_arrays_of_any_alignment(ctx, m, n, L, shift, ids, route):
    """Rows of every alignment, the array starting `shift` entries after 16 aligned bytes, guard ids around it."""
    import torch
    b = ballots(np.random.default_rng(m + shift), n, m, L, 0.3, ids)
    flat = np.full(b.size + 32, 1, dtype=b.dtype)
    flat[shift:shift + b.size] = b.reshape(-1)
    t = torch.from_numpy(flat).cuda()[shift:shift + b.size].view(n, L)
    ctx.set_sparse_count(route)
    try:
        d = ctx.pairwise(t, m)
    finally:
        ctx.set_sparse_count("bucketed")
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b, m, None))
