"""The merge of split-key partials at its edges: 2 .. 64 splits (rounds of eight, the narrow and the wide form), waves whose
rows belong to several requests (two query heads, one token each, requests without tokens between them), both head sizes."""
import numpy as np
import pytest
import torch

from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,n_q,kv_len", [
    (128, [1], [130]),                                     # two or three splits
    (128, [3], [64 * 8 + 5]),                              # a second round with one split
    (64, [2], [64 * 17]),                                  # a third round, statistics past one per lane
    (128, [1, 2, 0, 1, 1, 3], [70, 900, 64, 640, 2100, 64 * 64]),
    (64, [1, 1, 1, 0, 0, 1, 2, 1, 1], [200, 64 * 33, 65, 64, 64, 1000, 64 * 64 + 9, 3, 400]),
])
def test_merge_of_splits(head_dim, n_q, kv_len):
    """Positions are 0, so nothing is rotated and the result is a plain softmax over the rows, taken in fp64.  Bound: the
    relative error of bf16 queries, weights and results, 1e-2 as for every bf16 attention here (3e-3 is what they show)."""
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(2, 1, head_dim, "bf16", 1e4, 0))
    g = torch.Generator().manual_seed(head_dim + len(n_q))
    start = np.concatenate([[0], np.cumsum(kv_len)]).astype(np.int64)
    cu = np.concatenate([[0], np.cumsum(n_q)]).astype(np.int32)
    q = torch.randn(int(cu[-1]), 2, head_dim, generator=g).bfloat16()
    k, v = (torch.randn(int(start[-1]), 1, head_dim, generator=g).bfloat16() for _ in range(2))
    out = torch.full_like(q, float("nan")).cuda()
    B.tr_set_tuning("min_split_keys", 64)
    B.tr_set_tuning("target_items", 1024)
    try:
        ws = B.workspace(B.tr_prefill_attn_batched_workspace_size(gs, cu, start))
        assert ws is not None and ws.numel() > 256
        B.tr_prefill_attn_batched(gs, q.cuda(), k.cuda(), v.cuda(), torch.zeros(int(cu[-1]), dtype=torch.int32).cuda(), cu, start, out, ws)
        torch.cuda.synchronize()
    finally:
        B.tr_set_tuning("min_split_keys", 0)
        B.tr_set_tuning("target_items", 0)
    for r, (n, kv) in enumerate(zip(n_q, kv_len)):
        for i in range(n):
            keys = slice(int(start[r]), int(start[r]) + kv - n + i + 1)
            s = q[cu[r] + i].double() @ k[keys, 0].double().T / head_dim ** 0.5
            want = torch.softmax(s, 1) @ v[keys, 0].double()
            got = out[cu[r] + i].cpu().double()
            assert (got - want).norm() < 1e-2 * want.norm(), (r, i)
