"""Every width class of the row kernels against the oracle: rows of one to
64 lanes (the group sums of dot products and squared norms cross lanes in a
different way in each), and widths at the edges of each class."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2206_00470_amd import Store
from paper_2206_00470_amd.workloads import (CTR_33M, KGE_COMPLEX, MF_10Mx1M, SGNS_1M, CTRWorkload, KGEWorkload,
                                            MFWorkload, SGNSWorkload, small_variant)
from tests.helpers import assert_close_tables, say

pytestmark = pytest.mark.gpu

DIMS = [4, 8, 12, 16, 20, 28, 32, 36, 64, 68, 100, 128, 132, 256, 260, 384, 512]   # four floats per lane
DIMS += [1, 2, 13, 50, 63, 65, 127, 129, 255, 257, 511]                             # one float per lane


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def tables(K, d, rowwise, seed):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((K, d), dtype=np.float32) * np.float32(0.1))
    G = rng.uniform(0.05, 1, K if rowwise else (K, d)).astype(np.float32)
    return W, G


def check(what, Wt, Gt, W, G, loss, rloss):
    Gg = Gt.cpu().numpy()
    assert_close_tables(Wt.cpu().numpy(), W, f"{what} W")
    assert_close_tables(Gg.reshape(len(G), -1), G.reshape(len(G), -1), f"{what} G")
    assert float(loss.item()) == pytest.approx(rloss, rel=1e-9)


@pytest.mark.parametrize("rowwise", [False, True], ids=["element", "rowwise"])
@pytest.mark.parametrize("dim", DIMS)
def test_steps_of_every_row_width(dim, rowwise):
    lr, eps = 0.1, 1e-10
    mf = replace(small_variant(MF_10Mx1M), rank=dim, n_rows=900, n_cols=300, batch=1501)
    b = MFWorkload(mf).batch(0)
    say(f"dim {dim} {'row-wise' if rowwise else 'per element'}: mf")
    W, G = tables(mf.num_keys, dim, rowwise, dim)
    Wt, Gt = dev(W), dev(G)
    s = Store(Wt, Gt, lr, eps)
    loss = s.step_mf(dev(b.row), dev(b.col), dev(b.val), mf.n_rows, mf.lam)
    assert s.error() == 0
    args = (b.row, b.col, b.val, mf.n_rows, mf.lam)
    rloss = (oracle.step_rowwise("mf", W, G, args, lr, eps) if rowwise else oracle.step_mf(W, G, *args, lr, eps))[0]
    check("mf", Wt, Gt, W, G, loss, rloss)

    sg = replace(small_variant(SGNS_1M), dim=dim, vocab=500, batch=67, n_neg=5)
    b = SGNSWorkload(sg).batch(0)
    say("  sgns")
    W, G = tables(sg.num_keys, dim, rowwise, dim + 1)
    Wt, Gt = dev(W), dev(G)
    s = Store(Wt, Gt, lr, eps)
    loss = s.step_sgns(dev(b.centre), dev(b.ctx), dev(b.neg), sg.window, sg.vocab)
    assert s.error() == 0
    args = (b.centre, b.ctx, b.neg, sg.window, sg.vocab)
    rloss = (oracle.step_rowwise("sgns", W, G, args, lr, eps) if rowwise else oracle.step_sgns(W, G, *args, lr, eps))[0]
    check("sgns", Wt, Gt, W, G, loss, rloss)

    ct = replace(small_variant(CTR_33M), dim=dim, n_fields=7, batch=93, table_rows=2000)
    b = CTRWorkload(ct).batch(0)
    say("  ctr")
    W, G = tables(ct.num_keys, dim, rowwise, dim + 2)
    Wt, Gt = dev(W), dev(G)
    s = Store(Wt, Gt, lr, eps)
    loss = s.step_ctr(dev(b.keys), dev(b.label))
    assert s.error() == 0
    rloss = (oracle.step_rowwise("ctr", W, G, (b.keys, b.label), lr, eps) if rowwise
             else oracle.step_ctr(W, G, b.keys, b.label, lr, eps))[0]
    check("ctr", Wt, Gt, W, G, loss, rloss)

    if dim % 2:
        return                     # ComplEx rows are pairs
    kg = replace(small_variant(KGE_COMPLEX), cdim=dim // 2, n_ent=700, n_rel=11, batch=41, n_triples=410, n_neg=14,
                 n_head_neg=7)
    b = KGEWorkload(kg).batch(0)
    say("  kge")
    W, G = tables(kg.num_keys, dim, rowwise, dim + 3)
    Wt, Gt = dev(W), dev(G)
    s = Store(Wt, Gt, lr, eps)
    loss = s.step_kge(dev(b.head), dev(b.rel), dev(b.tail), dev(b.neg), kg.n_head_neg, kg.n_ent)
    assert s.error() == 0
    args = (b.head, b.rel, b.tail, b.neg, kg.n_head_neg, kg.n_ent)
    rloss = (oracle.step_rowwise("kge", W, G, args, lr, eps) if rowwise else oracle.step_kge(W, G, *args, lr, eps))[0]
    check("kge", Wt, Gt, W, G, loss, rloss)
