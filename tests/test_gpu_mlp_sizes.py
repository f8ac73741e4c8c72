"""Network kernels at the edges of their tiles (64 rows), workgroups and
segment registers, against the float64 network."""
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


@pytest.mark.parametrize("sizes", [[1], [63], [64], [65, 1], [1, 0, 2], [2047, 2048, 2049], [300] * 60])
def test_loss_and_gradient(ctx, sizes):
    import torch
    rng = np.random.default_rng(sum(sizes))
    M = sum(sizes)
    X = rng.standard_normal((M, 16)).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    win = np.zeros(M, dtype=np.uint8)
    for a, b in zip(off[:-1], off[1:]):
        if b > a and (b - a) % 7 != 5:
            win[rng.integers(a, b)] = 1
    p = omlp.init_params(3)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    s = ctx.mlp_forward(t(p), t(X))
    ds, loss = ctx.mlp_loss(s, t(off), t(win))
    grad = ctx.mlp_backward(t(p), t(X), ds).cpu().numpy()
    want_s = omlp.forward(p, X, rounding=True)["s"]
    assert np.linalg.norm(s.cpu().numpy() - want_s) <= 1e-2 * np.linalg.norm(want_s)
    s64 = s.cpu().numpy().astype(np.float64)
    want_loss, want_ds = omlp.seg_loss(s64, off, win, np.float64)
    assert abs(float(loss.double().sum()) / len(sizes) - want_loss) <= 1e-5 * max(1.0, abs(want_loss))
    assert np.abs(ds.cpu().numpy() - want_ds).max() <= 1e-6
    want = omlp.backward(p, X, ds.cpu().numpy(), rounding=True)
    assert np.linalg.norm(grad - want) <= 1e-2 * max(np.linalg.norm(want), 1e-12)

