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


@pytest.mark.parametrize("ids", ["u16", "i32"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("m,n,L,cut", [
    (1, 5, 1, 0.5), (2, 33, 2, 0.5), (3, 32, 2, 0.0), (17, 31, 16, 0.3), (64, 65, 64, 0.0), (65, 1, 65, 0.0),
    (127, 97, 127, 0.4), (128, 64, 127, 0.4), (129, 600, 129, 0.2), (255, 40, 7, 0.5), (257, 2000, 256, 0.5),
    (1025, 70, 1025, 0.3), (2049, 33, 2049, 0.1), (1100, 3000, 9, 0.2), (700, 999, 699, 1.0)])
def test_counts(ctx, m, n, L, cut, weighted, ids):
    import torch
    rng = np.random.default_rng(m * 1000 + n)
    b = ballots(rng, n, m, L, cut, ids)
    w = rng.integers(0, 1 << 20 if m % 2 else 41, size=n).astype(np.uint32) if weighted else None
    d = ctx.pairwise(torch.from_numpy(b).cuda(), m, dtype="i32",
                     voter_weight=None if w is None else torch.from_numpy(w).cuda())
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
