"""Bucketed counting of truncated ballots, with the route asserted: rows of
every length around the steps they are read in, candidates with several items,
repeated ids, and outputs of any pitch whose padding stays as it was."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CT = 128


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


def rank_bits(last):
    b = 1
    while (1 << b) - 1 < last:
        b += 1
    return b


def takes_buckets(b, m, weighted):
    """Whether the device counts these truncated ballots by pairs: the rule of
    the route decision.  (m above the one-pass count's limit.)"""
    assert 4096 < m <= 32768 and b.size <= 1 << 27
    if weighted:
        return True
    listed = np.where((b < 0).any(1), (b < 0).argmax(1), b.shape[1])
    assert listed.max() < m - 1
    nu = len(np.unique(b[b >= 0]))
    pitch = (nu + 1 + CT - 1) // CT * CT
    bits = rank_bits(b.shape[1] if b.shape[1] <= 64 else listed.max())
    groups = -(-len(b) // 32)
    dense = groups * pitch * pitch * (bits + 2) / 45.0 + 3.0 * m * m
    return dense > 6.0 * (listed * (listed - 1) // 2).sum() + m * m


def count(ctx, b, m, w, ids, dtype, out=None):
    import torch
    x = np.where(b < 0, 0xFFFF, b).astype(np.uint16) if ids == "u16" else b
    ctx.reset_timing()
    ctx.set_timing(True)
    d = ctx.pairwise(torch.from_numpy(x).cuda(), m, voter_weight=None if w is None else torch.from_numpy(w).cuda(),
                     dtype=dtype, out=out)
    torch.cuda.synchronize()
    ctx.set_timing(False)
    # bucket count, columns, scan, placement, accumulation (one launch of the atomic route instead)
    assert ctx.kernel_time("route")[0] == (1 if w is None else 2) and ctx.kernel_time("count_sparse")[0] == 5
    return d


def ballots(rng, n, L, m, popular=0):
    """n ballots of up to L distinct ids (the last one full), the first `popular` ids on every long enough one."""
    b = np.full((n, L), -1, dtype=np.int32)
    for i in range(n):
        ids = rng.permutation(np.concatenate([np.arange(popular), popular + rng.choice(m - popular, L, False)])[:L])
        k = L if i == n - 1 else rng.integers(0, L + 1)
        b[i, :k] = ids[:k]
    return b


KINDS = [("u16", False, "u16"), ("i32", False, "i32"), ("u16", True, "i32"), ("i32", True, "i32"), ("i32", True, "u16")]


@pytest.mark.parametrize("ids,weighted,dtype", KINDS)
@pytest.mark.parametrize("L", [15, 16, 17, 32, 33, 48, 49, 64, 65, 66, 96, 97, 98, 128, 129, 130, 161, 200])
def test_row_lengths(ctx, L, ids, weighted, dtype):
    rng = np.random.default_rng(L)
    m, n = 4500, 130
    b = ballots(rng, n, L, m, 2)
    b[:8, :] = b[-1, rng.permutation(L)]  # full rows among the first ones too
    w = rng.integers(0, 9, size=n).astype(np.uint32) if weighted else None
    assert takes_buckets(b, m, weighted)
    d = count(ctx, b, m, w, ids, dtype)
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b, m, w))


@pytest.mark.parametrize("ids,weighted,dtype", KINDS)
@pytest.mark.parametrize("L", [9, 40, 70])
def test_candidates_of_several_items(ctx, L, ids, weighted, dtype):
    # items hold 1024 occurrences here (the smallest bound: few occurrences per workgroup)
    rng = np.random.default_rng(100 + L)
    m, n = 4500, 4300
    many = (n, 2500, 1500, 1025, 1024)  # id c on the first many[c] ballots
    b = np.full((n, L), -1, dtype=np.int32)
    for i in range(n):
        ids_i = [c for c in range(5) if i < many[c]]
        ids_i += list(5 + rng.choice(m - 5, (L if i == 0 else rng.integers(len(ids_i), L + 1)) - len(ids_i), False))
        b[i, :len(ids_i)] = rng.permutation(ids_i)
    items = -(-np.bincount(b[b >= 0], minlength=m) // 1024)
    assert list(items[:5]) == [5, 3, 2, 2, 1] and items[5:].max() == 1
    w = rng.integers(0, 3, size=n).astype(np.uint32) if weighted else None
    assert takes_buckets(b, m, weighted)
    d = count(ctx, b, m, w, ids, dtype)
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b, m, w))


@pytest.mark.parametrize("ids,weighted,dtype", KINDS)
@pytest.mark.parametrize("L", [9, 40, 70, 150])
@pytest.mark.parametrize("first,second", [(0, 1), (2, 7), (0, -1), (-2, -1)])
def test_repeated_id(ctx, L, first, second, ids, weighted, dtype):
    import paper_2505_12976_amd as sz
    m, n = 4500, 130
    b = ballots(np.random.default_rng(L), n, L, m, 2)
    w = np.ones(n, dtype=np.uint32) if weighted else None
    b[n - 1, first] = b[n - 1, second]  # (the ballot that is full)
    count(ctx, b, m, w, ids, dtype)
    assert ctx.device_error() == sz.EBALLOT
    b[n - 1, second % L:] = -1
    assert takes_buckets(b, m, weighted)
    d = count(ctx, b, m, w, ids, dtype)
    assert ctx.device_error() == 0
    assert np.array_equal(d.cpu().numpy().astype(np.int64), oracle.pairwise(b, m, w))
