"""The skip-gram step at the edges of its row tiles, against the oracle: fewer
rows than one batch of four, whole tiles and remainders, more than 64 slots,
absent slots, and scores that saturate the sigmoid, in row groups of 4, 32 and
64 lanes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2206_00470_amd import Store
from tests.helpers import assert_close_tables, say

pytestmark = pytest.mark.gpu

# window, negatives: 2, 2 x 3, 63 + 1, 64 + 4 and 10 x 26 rows; 66 slots of one row
SIZES = [(1, 0), (1, 2), (2, 15), (2, 16), (5, 25), (33, 0)]


@pytest.mark.parametrize("scale", [0.1, 2.0], ids=["ordinary", "saturated"])
@pytest.mark.parametrize("dim", [16, 100, 300, 13])
@pytest.mark.parametrize("window,neg", SIZES)
def test_sgns_tiles(window, neg, dim, scale):
    V, B, lr, eps = 700, 45, 0.1, 1e-10
    say(f"sgns tiles: window {window} neg {neg} dim {dim} scale {scale}")
    rng = np.random.default_rng(1000 * window + 10 * neg + dim)
    W = (rng.standard_normal((2 * V, dim)) * scale).astype(np.float32)
    G = rng.uniform(0.05, 1, W.shape).astype(np.float32)
    centre = rng.integers(0, V, B).astype(np.int32)
    ctx = rng.integers(0, V, (B, 2 * window)).astype(np.int32)
    ctx[rng.random(ctx.shape) < 0.3] = -1
    ctx[0] = -1                      # a centre without rows
    ctx[1] = rng.integers(0, V, 2 * window)
    ng = rng.integers(0, V, (B, 2 * window, neg)).astype(np.int32)
    ng[ctx < 0] = -1
    Wt, Gt = torch.from_numpy(W.copy()).cuda(), torch.from_numpy(G.copy()).cuda()
    s = Store(Wt, Gt, lr, eps)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    loss = s.step_sgns(dev(centre), dev(ctx), dev(ng), window, V)
    assert s.error() == 0
    rloss, bad = oracle.step_sgns(W, G, centre, ctx, ng, window, V, lr, eps)
    assert bad == 0
    assert_close_tables(Wt.cpu().numpy(), W, "W")
    assert_close_tables(Gt.cpu().numpy(), G, "G")
    assert float(loss.item()) == pytest.approx(rloss, rel=1e-9)


@pytest.mark.parametrize("value", [np.inf, -np.inf, 3e38], ids=["inf", "-inf", "large"])
@pytest.mark.parametrize("dim", [16, 100, 300, 13])
@pytest.mark.parametrize("window,neg", [(1, 0), (1, 2), (2, 16), (33, 0)])
def test_infinite_centre_and_absent_rows(window, neg, dim, value):
    """A centre row with an infinite element, in batches of four rows that are
    not all there (past the last row, or of an absent slot): the gradient of
    the centre is the sum over the rows that are, and finite."""
    V, lr, eps = 700, 0.1, 1e-10
    say(f"sgns infinite centre: window {window} neg {neg} dim {dim} value {value}")
    rng = np.random.default_rng(1000 * window + 10 * neg + dim)
    W = (rng.standard_normal((2 * V, dim)) * 0.1).astype(np.float32)
    G = rng.uniform(0.05, 1, W.shape).astype(np.float32)
    centre = np.array([5, 9, 11], dtype=np.int32)
    W[5, dim // 2] = value
    words = 20 + rng.permutation(V - 20)       # every output row once, so no infinities of either sign meet
    per = 2 * window * (1 + neg)
    ids = words[:3 * per].reshape(3, 2 * window, 1 + neg).astype(np.int32)
    ctx, ng = ids[:, :, 0].copy(), ids[:, :, 1:].copy()
    ctx[:2, 1] = -1
    ng[ctx < 0] = -1
    Wt, Gt = torch.from_numpy(W.copy()).cuda(), torch.from_numpy(G.copy()).cuda()
    s = Store(Wt, Gt, lr, eps)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    s.step_sgns(dev(centre), dev(ctx), dev(ng), window, V)
    assert s.error() == 0
    _, bad = oracle.step_sgns(W, G, centre, ctx, ng, window, V, lr, eps)
    assert bad == 0
    assert np.isfinite(G[5]).all()
    np.testing.assert_allclose(Gt.cpu().numpy(), G, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(Wt.cpu().numpy(), W, rtol=1e-5, atol=1e-6)
