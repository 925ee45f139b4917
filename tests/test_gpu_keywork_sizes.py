"""The key work (sort and segments) at the edges of its size classes: one
workgroup with 1, 4 or 8 keys per thread, tiles of 4,096 keys, and the
separate kernels above; with one to four radix passes, invalid keys, and keys
that are all the same (segments cut into chunks)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2206_00470_amd import Store, dedup
from tests.helpers import assert_close_tables, say

pytestmark = pytest.mark.gpu

SMALL = [1, 2, 63, 64, 65, 1023, 1024, 1025, 4095, 4096, 4097, 8191, 8192]
MID = [8193, 12288, 12289, 65537, 200_001, 96 * 4096 - 1, 96 * 4096]
ABOVE = [96 * 4096 + 1]


@pytest.mark.parametrize("num_keys", [2, 300, 70_000, 9_000_000, 2**31 - 1])
@pytest.mark.parametrize("n", SMALL + MID + ABOVE)
def test_dedup_sizes(n, num_keys):
    say(f"dedup n {n} num_keys {num_keys}")
    rng = np.random.default_rng(n + num_keys)
    keys = rng.integers(0, num_keys, n)
    keys[rng.random(n) < 0.3] = num_keys // 2     # a hot key
    keys[rng.random(n) < 0.05] = -1               # invalid ones sort last
    keys[rng.random(n) < 0.05] = num_keys
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    uniq, perm, offs, U = dedup(num_keys, torch.from_numpy(keys).cuda(), err=err)
    bad = (keys < 0) | (keys >= num_keys)
    order = np.argsort(np.where(bad, num_keys, keys), kind="stable")
    ru, start = np.unique(keys[order][:n - bad.sum()], return_index=True)
    assert U == len(ru)
    np.testing.assert_array_equal(uniq.cpu().numpy(), ru)
    np.testing.assert_array_equal(perm.cpu().numpy(), order)
    np.testing.assert_array_equal(offs.cpu().numpy(), np.append(start, n - bad.sum()))
    assert int(err.item()) == int(bad.any())


@pytest.mark.parametrize("kind", ["mixed", "one_column", "all_invalid"])
@pytest.mark.parametrize("B", [1, 500, 2047, 4096, 4097, 30_000, 196_609])
def test_mf_step_sizes(B, kind):
    """The split between row and column keys, whoever writes it."""
    say(f"mf B {B} {kind}")
    rows, cols, d, lr, eps = 3000, 700, 8, 0.1, 1e-10
    rng = np.random.default_rng(B)
    W = (rng.standard_normal((rows + cols, d)) * 0.1).astype(np.float32)
    G = rng.uniform(0.05, 1, W.shape).astype(np.float32)
    row = rng.integers(0, rows, B).astype(np.int32)
    col = rng.integers(0, cols, B).astype(np.int32)
    if kind == "one_column":
        col[:] = cols - 1
    elif kind == "all_invalid":
        col[:] = cols
    else:
        row[rng.random(B) < 0.1] = -1 if B > 1 else 0
    val = rng.standard_normal(B).astype(np.float32)
    dev = lambda a: torch.from_numpy(a.copy()).cuda()  # noqa: E731
    Wt, Gt = dev(W), dev(G)
    s = Store(Wt, Gt, lr, eps)
    loss = s.step_mf(dev(row), dev(col), dev(val), rows, 1e-2)
    rloss, bad = oracle.step_mf(W, G, row, col, val, rows, 1e-2, lr, eps)
    assert (s.error() != 0) == (bad != 0)
    assert_close_tables(Wt.cpu().numpy(), W, "W")
    assert_close_tables(Gt.cpu().numpy(), G, "G")
    assert float(loss.item()) == pytest.approx(rloss, rel=1e-9, abs=0.0 if kind != "all_invalid" else 1e-300)
