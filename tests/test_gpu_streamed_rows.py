"""The merge on both sides of the line where it streams table and gradient
rows past the caches (rows it can touch above 256 MB): each store layout
against the oracle, and equal bits on either side for the keys in common."""
import numpy as np
import pytest
import torch

import oracle
from paper_2206_00470_amd import Store
from tests.helpers import assert_bitwise, assert_close_tables, say

pytestmark = pytest.mark.gpu

LR, EPS = 0.1, 1e-10
LINE = 256 << 20   # bytes of value and accumulator rows


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("kind,dim,row_bytes", [("element", 512, 4096), ("element", 509, 4072), ("rowwise", 512, 2052),
                                                ("bf16", 512, 3072), ("bf16", 511, 3066)])
def test_push_around_the_streaming_line(kind, dim, row_bytes):
    n_line = LINE // row_bytes            # the last size that is not streamed
    K = n_line + 300
    rng = np.random.default_rng(dim)
    W = (rng.standard_normal((K, dim), dtype=np.float32) * np.float32(0.1))
    G = rng.uniform(0.05, 1, K if kind == "rowwise" else (K, dim)).astype(np.float32)
    keys = rng.permutation(K)[:n_line + 1].astype(np.int64)
    keys[-200:] = keys[0]                 # one segment long enough to be cut
    grads = rng.standard_normal((n_line + 1, dim), dtype=np.float32)
    got = []
    for n in (n_line, n_line + 1):
        say(f"push {kind} dim {dim} n {n}")
        if kind == "bf16":
            Wt = dev(oracle.f32_to_bf16(W).view(np.int16)).view(torch.bfloat16)
        else:
            Wt = dev(W)
        Gt = dev(G)
        s = Store(Wt, Gt, LR, EPS)
        s.push(dev(keys[:n]), dev(grads[:n]))
        assert s.error() == 0
        Wg = (Wt.view(torch.int16) if kind == "bf16" else Wt).cpu().numpy()
        got.append((Wg, Gt.cpu().numpy()))
        s.close()
    hot = keys[0]
    rest = np.setdiff1d(np.arange(K), [hot])
    for a, b, what in zip(got[0], got[1], ("W", "G")):
        assert_bitwise(a[rest], b[rest], f"{what} rows of the keys in common")
    Wr, Gr = (oracle.f32_to_bf16(W) if kind == "bf16" else W.copy()), G.copy()
    {"element": oracle.push, "rowwise": oracle.push_rowwise, "bf16": oracle.push_bf16}[kind](
        Wr, Gr, keys, grads, LR, EPS)
    Wg = got[1][0]
    if kind == "bf16":
        Wg, Wr = oracle.bf16_to_f32(Wg.view(np.uint16)), oracle.bf16_to_f32(Wr)
    assert_close_tables(Wg, Wr, "W")
    assert_close_tables(got[1][1], Gr, "G")
