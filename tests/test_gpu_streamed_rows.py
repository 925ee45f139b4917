"""The merge on both sides of the line where it streams table and gradient
rows past the caches (rows it can touch above 256 MB; rows of one float per
lane only in row-wise stores, both sides cached otherwise): each store layout's
push and each task's step against the oracle, and equal bits on either side
for the keys in common."""
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


@pytest.mark.parametrize("kind,dim,row_bytes", [("element", 512, 4096), ("element", 509, 4072), ("rowwise", 512, 2052), ("rowwise", 511, 2048),
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


def batch(task, K, n, rng):
    """Arguments of a step of a little over n occurrences over K keys."""
    i32 = lambda *a: rng.integers(*a).astype(np.int32)  # noqa: E731
    if task == "mf":
        B, cols = n // 2 + 8, 1000
        col = i32(0, cols, B)
        col[: B // 4] = 3                                  # a hot column
        return (i32(0, K - cols, B), col, rng.standard_normal(B).astype(np.float32), K - cols, 1e-2)
    if task == "kge":
        neg, rels = 62, 20
        B = n // (3 + neg) + 2
        return i32(0, K - rels, B), i32(0, rels, B), i32(0, K - rels, B), i32(0, K - rels, (B, neg)), neg // 2, K - rels
    if task == "sgns":
        w, neg, V = 3, 10, K // 2
        B = n // (1 + 2 * w * (1 + neg)) + 2
        ctx, ng = i32(0, V, (B, 2 * w)), i32(0, V, (B, 2 * w, neg))
        ctx[rng.random(ctx.shape) < 0.1] = -1
        ng[ctx < 0] = -1
        ng[:, :, 0][ctx >= 0] = 7                          # a hot output word
        return i32(0, V, B), ctx, ng, w, V
    F = 26
    B = n // F + 2
    return rng.integers(0, K, (B, F)), (rng.random(B) < 0.25).astype(np.float32)


@pytest.mark.parametrize("task,dim,rowwise", [
    ("mf", 512, False), ("mf", 512, True), ("kge", 512, False), ("kge", 512, True), ("kge", 510, False),
    ("sgns", 512, False), ("sgns", 512, True), ("sgns", 509, False), ("kge", 510, True), ("sgns", 509, True), ("ctr", 512, False), ("ctr", 512, True)])
def test_steps_around_the_streaming_line(task, dim, rowwise):
    """The same batch on a table of as many rows as are not streamed, and on
    one of a single row more: equal bits, and the oracle's step."""
    K = LINE // (4 * dim + (4 if rowwise else 4 * dim))
    K -= task == "sgns" and K % 2
    rng = np.random.default_rng(dim)
    W = (rng.standard_normal((K + 2, dim), dtype=np.float32) * np.float32(0.1))
    G = rng.uniform(0.05, 1, K + 2 if rowwise else (K + 2, dim)).astype(np.float32)
    args = batch(task, K, K + 2, rng)
    put = lambda a: dev(a) if isinstance(a, np.ndarray) else a  # noqa: E731
    got = []
    for rows in (K, K + 2):
        say(f"{task} dim {dim} rowwise {rowwise} rows {rows}")
        Wt, Gt = dev(W[:rows]), dev(G[:rows])
        s = Store(Wt, Gt, LR, EPS)
        loss = getattr(s, f"step_{task}")(*map(put, args))
        assert s.error() == 0
        got.append((Wt.cpu().numpy(), Gt.cpu().numpy(), float(loss.item())))
        s.close()
    assert_bitwise(got[0][0], got[1][0][:K], "W")
    assert_bitwise(got[0][1], got[1][1][:K], "G")
    assert got[0][2] == got[1][2]
    rloss, bad = (oracle.step_rowwise(task, W, G, args, LR, EPS) if rowwise
                  else getattr(oracle, f"step_{task}")(W, G, *args, LR, EPS))
    assert bad == 0
    assert_close_tables(got[1][0], W, "W")
    assert_close_tables(got[1][1].reshape(K + 2, -1), G.reshape(K + 2, -1), "G")
    assert got[1][2] == pytest.approx(rloss, rel=1e-9)
