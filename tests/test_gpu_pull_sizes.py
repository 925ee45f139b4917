"""Pulls at the edges of their launch: rows of every lane layout, counts that
give groups one, three and four rows, outputs below and above the size that is
written past the caches, and outputs that are not 16-byte aligned."""
import numpy as np
import pytest
import torch

from paper_2206_00470_amd import Store
from paper_2206_00470_amd.store import interleaved_bf16_tables
from tests.helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("dim", [4, 13, 64, 100, 256, 300, 512])
@pytest.mark.parametrize("n", [1, 5, 63, 1027, "one row", "four rows", "large", "streamed"])
def test_pull_sizes(n, dim, bf16):
    lanes = 64 if dim % 4 else next(x for x in (4, 8, 16, 32, 64) if 4 * x >= dim or x == 64)
    if n in ("one row", "four rows"):   # the last count with one row per group, the first ones with three and four
        n = 2048 * (256 // lanes) + (0 if n == "one row" else 5)
    elif n == "large":
        n = (32 << 20) // (4 * dim) + 3
    elif n == "streamed":
        n = (256 << 20) // (4 * dim) + 3
    say(f"pull n {n} dim {dim} bf16 {bf16}")
    K = 5000
    rng = np.random.default_rng(dim)
    W0 = torch.from_numpy(rng.standard_normal((K, dim)).astype(np.float32)).cuda()
    W, G = interleaved_bf16_tables(W0, torch.zeros_like(W0)) if bf16 else (W0, torch.zeros_like(W0))
    s = Store(W, G, 0.1, 1e-10)
    keys = torch.from_numpy(rng.integers(0, K, n)).cuda()
    keys[0] = K - 1
    bad = n // 2 if n > 1 else None
    if bad:
        keys[bad] = K + 7          # a key out of range pulls zeros
    want = W.float()[keys.clamp(max=K - 1)]
    if bad:
        want[bad] = 0
    big = torch.full((n * dim + 1 + 64,), 7.5, device="cuda")
    for shift in (0, 1):           # aligned, and 4 bytes past
        out = big[shift:shift + n * dim].view(n, dim)
        s.pull(keys, out=out)
        assert torch.equal(out, want)
        assert bool((big[shift + n * dim:] == 7.5).all())
        big.fill_(7.5)
    assert (s.error() != 0) == (bad is not None)
