"""Bucketed counting of truncated ballots: items of one candidate's
occurrences at their edges (less ballots than one 16-byte piece of ids, the
last piece of the array, ballots longer than the ids in flight, candidates
with several items, both LDS rows, rows that end inside a store)."""
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


def ballots(n, L, m, popular, seed):
    """n ballots of 1 .. L distinct ids; `popular` of the ids are on most of them."""
    rng = np.random.default_rng(seed)
    b = np.full((n, L), -1, dtype=np.int32)
    for i in range(n):
        head = rng.permutation(popular)[:rng.integers(0, popular + 1)] if popular else np.empty(0, np.int64)
        tail = popular + rng.permutation(m - popular)[:L]
        ids = rng.permutation(np.concatenate([head, tail])[:L])
        b[i, :len(ids)] = ids
        b[i, rng.integers(1, L + 1):] = -1
    b[-1, :] = rng.permutation(m)[:L]  # the last ballot is full: its ids end the array
    return b


@pytest.mark.parametrize("n,L,m,popular", [
    (1, 3, 4999, 0),       # less than one piece in all
    (2, 4, 4999, 0),       # exactly one piece of uint16 ids
    (3, 7, 5003, 0),       # pieces at every offset
    (700, 45, 4998, 3),    # longer than the ids in flight
    (2600, 9, 5001, 2),    # candidates with two and three items
    (40, 150, 16500, 1),   # the larger LDS row
])
@pytest.mark.parametrize("ids", ["u16", "i32"])
@pytest.mark.parametrize("weighted,dtype", [(False, "u16"), (False, "i32"), (True, "i32")])
def test_occurrence_items(ctx, n, L, m, popular, ids, weighted, dtype):
    import torch
    b = ballots(n, L, m, popular, 31 * n + L)
    weight = np.random.default_rng(n).integers(0, 5, size=n).astype(np.uint32) if weighted else None
    want = oracle.pairwise(b, m, weight)
    if ids == "u16":
        t = torch.from_numpy(np.where(b < 0, 0xFFFF, b).astype(np.uint16)).to("cuda:0")
    else:
        t = torch.from_numpy(b).to("cuda:0")
    wt = None if weight is None else torch.from_numpy(weight.astype(np.int64)).to(torch.uint32).to("cuda:0")
    d = ctx.pairwise(t, m, voter_weight=wt, dtype=dtype)
    torch.cuda.synchronize()
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), want)
