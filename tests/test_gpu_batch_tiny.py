"""Thousands of tiny elections whose counts and closures lie next to each other
in the same cache lines, replayed with other ballots in the same buffers: every
replay against the oracle."""
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


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("topk", [0, 2])
def test_tiny_elections(ctx, topk, graph):
    import torch
    from paper_2505_12976_amd import batch as zb
    rng = np.random.default_rng(11 + topk)
    sizes = [(int(rng.integers(1, 13)), int(rng.integers(1, 70))) for _ in range(2500)]
    sizes += [(int(rng.integers(90, 200)), 40) for _ in range(20)]  # several count items among them
    rng.shuffle(sizes)

    def draw():
        return [np.argsort(rng.random((n, m)), axis=1)[:, :max(1, m - 2 * (m % 2))].astype(np.uint16) for m, n in sizes]

    ms = [m for m, _ in sizes]
    packed = zb.pack(draw(), ms, np.uint16)
    ballots = torch.from_numpy(packed.ballots).cuda()
    out = zb.alloc_outputs(packed, "cuda:0")
    level = torch.empty_like(out["order"]) if topk else None
    plan = ctx.batch_plan(packed.elections, "u16", topk=topk)
    try:
        for _ in range(3):
            profiles = draw()
            ballots.copy_(torch.from_numpy(zb.pack(profiles, ms, np.uint16).ballots))
            for t in out.values():
                t.fill_(77)
            ctx.batch_run(plan, ballots, out["d"], out["is_winner"], p=out["p"], n_winners=out["n_winners"],
                          beaten_by=out["beaten_by"], order=out["order"], graph=graph, level=level)
            torch.cuda.synchronize()
            assert ctx.device_error() == 0
            host = {k: t.cpu() for k, t in out.items()}
            levels = level.cpu() if topk else None
            for e, m in enumerate(ms):
                want = oracle.schulze(profiles[e], m, oracle.WINNING_VOTES)
                assert np.array_equal(packed.mat(host["d"], e).numpy(), want["d"]), e
                assert np.array_equal(packed.mat(host["p"], e).numpy(), want["p"]), e
                assert np.array_equal(packed.vec(host["is_winner"], e).numpy() != 0, want["is_winner"]), e
                assert np.array_equal(packed.vec(host["order"], e).numpy(), want["order"]), e
                assert int(host["n_winners"][e]) == want["is_winner"].sum(), e
                if topk:
                    assert np.array_equal(packed.vec(levels, e).numpy() == 0, want["is_winner"]), e
    finally:
        plan.destroy()
