"""Weighted profiles with more than one fault: whichever way they are counted,
an id out of range is reported before a total weight of 2^32 or more, that
before a repeated id, and that before a count that does not fit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2505_12976_amd as sz
    c = sz.Context(0)
    yield c
    c.close()


# one pass over all candidates; full rankings and short ballots through the other routes
@pytest.mark.parametrize("m,n,L", [(40, 70, 40), (40, 70, 9), (4100, 70, 9), (4100, 70, 100)])
@pytest.mark.parametrize("faults,want", [
    ("range total repeat", "EBALLOT"), ("total repeat", "ERANGE"), ("range total", "EBALLOT"), ("total", "ERANGE"),
    ("repeat count", "EBALLOT"), ("count", "ERANGE"), ("", "OK")])
def test_first_error(ctx, m, n, L, faults, want):
    import torch
    import paper_2505_12976_amd as sz
    b = np.argsort(np.random.default_rng(L).random((n, m)), axis=1)[:, :L].astype(np.int32)
    w = np.ones(n, dtype=np.uint32)
    if "range" in faults:
        b[3, 4] = m
    if "repeat" in faults:
        b[37, 5] = b[37, 2]
    if "total" in faults:
        w[:] = 1 << 26
    if "count" in faults:
        b[:, 0], b[:, 1] = 1, 0  # everyone puts 1 first
        b[:, 2:] = 2 + np.argsort(np.random.default_rng(m).random((n, m - 2)), axis=1)[:, :L - 2]
        if "repeat" in faults:
            b[37, 5] = b[37, 2]
        w[:] = 2000
    ctx.pairwise(torch.from_numpy(b).cuda(), m, voter_weight=torch.from_numpy(w).cuda(), dtype="u16")
    assert ctx.device_error() == getattr(sz, want)
