"""The merge of split-key partials at its edges: 2 .. 64 splits (rounds of eight for a group of lanes, 32 and 64 statistics, a
wave for each row and D/8 lanes per row), waves whose rows belong to several requests (two query heads, one token each,
requests without tokens between them), both head sizes."""
import numpy as np
import pytest
import torch

from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def splits_of(nbytes, rows, head_dim):
    """How many key splits a workspace of one request with `rows` query rows is for."""
    up = lambda n: (n + 255) // 256 * 256
    n, = [s for s in range(2, 65) if up(s * rows * head_dim * 2) + up(s * rows * 8) == nbytes]
    return n


@pytest.mark.parametrize("head_dim,n_q,kv_len,wg_rows,splits", [
    # workgroups of 128 rows cut keys at multiples of 64, those of 32 rows (the choice for so few query rows) of 128
    (128, [1], [130], 0, 2),
    (128, [1], [130], 128, 3),
    (128, [3], [64 * 8], 128, 8),            # one round, full
    (128, [3], [64 * 8 + 5], 128, 9),        # a second round with one split
    (64, [2], [64 * 16], 128, 16),           # the most for which eight or sixteen lanes merge a row of these
    (64, [2], [64 * 17], 0, 9),
    (64, [2], [64 * 17], 128, 17),           # a wave per row from here on
    (128, [2], [64 * 33], 128, 33),
    (128, [5], [64 * 64], 128, 64),          # statistics for every lane
    (64, [5], [64 * 64], 128, 64),
    (64, [1], [64 * 61], 128, 61),
    (128, [1030], [64 * 20], 128, 20),       # 2060 rows: lanes again, three rounds
    (128, [1030], [64 * 49], 128, 49),       # and 64 statistics
    (64, [1030], [64 * 64], 128, 64),
    (128, [1, 2, 0, 1, 1, 3], [70, 900, 64, 640, 2100, 64 * 64], 0, None),
    (128, [1, 2, 0, 1, 1, 3], [70, 900, 64, 640, 2100, 64 * 64], 128, None),
    (128, [1, 2, 0, 1, 1, 3], [70, 900, 64, 640, 1020, 64 * 15], 128, None),   # the same requests, a few lanes per row
    (64, [1, 1, 1, 0, 0, 1, 2, 1, 1], [200, 64 * 33, 65, 64, 64, 1000, 64 * 64 + 9, 3, 400], 0, None),
    (64, [1, 1, 1, 0, 0, 1, 2, 1, 1], [200, 64 * 33, 65, 64, 64, 1000, 64 * 64, 3, 400], 128, None),
    (64, [1, 1, 1, 0, 0, 1, 2, 1, 1], [200, 64 * 13, 65, 64, 64, 1000, 64 * 11 + 9, 3, 400], 128, None),
])
def test_merge_of_splits(head_dim, n_q, kv_len, wg_rows, splits):
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
    B.tr_set_tuning("target_items", 4096)
    B.tr_set_tuning("wg_rows", wg_rows)
    try:
        need = B.tr_prefill_attn_batched_workspace_size(gs, cu, start)
        ws = B.workspace(need)
        assert splits is None or splits_of(need, 2 * n_q[0], head_dim) == splits
        assert ws is not None and ws.numel() > 256
        B.tr_prefill_attn_batched(gs, q.cuda(), k.cuda(), v.cuda(), torch.zeros(int(cu[-1]), dtype=torch.int32).cuda(), cu, start, out, ws)
        torch.cuda.synchronize()
    finally:
        for name in ("min_split_keys", "target_items", "wg_rows"):
            B.tr_set_tuning(name, 0)
    out = out.cpu().double()
    for r, (n, kv) in enumerate(zip(n_q, kv_len)):
        keys = slice(int(start[r]), int(start[r]) + kv)
        s = torch.matmul(q[cu[r]:cu[r + 1]].double().reshape(2 * n, head_dim), k[keys, 0].double().T) / head_dim ** 0.5
        hidden = torch.arange(kv)[None, :] > torch.arange(kv - n, kv).repeat_interleave(2)[:, None]
        want = torch.matmul(torch.softmax(s.masked_fill(hidden, float("-inf")), 1), v[keys, 0].double()).reshape(n, 2, head_dim)
        worst = ((out[cu[r]:cu[r + 1]] - want).norm(dim=-1) / want.norm(dim=-1)).reshape(-1)
        assert not worst.isnan().any() and (n == 0 or worst.max() < 1e-2), (r, int(worst.argmax()), float(worst.max()))
