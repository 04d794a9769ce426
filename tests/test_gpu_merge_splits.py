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
    (128, [3], [64 * 8], 128, 8),            # one round of eight or sixteen lanes, full
    (128, [3], [64 * 8 + 5], 128, 9),        # a wave per row from here on
    (64, [2], [64 * 17], 0, 9),
    (64, [2], [64 * 16], 128, 16),
    (64, [2], [64 * 17], 128, 17),
    (128, [512], [64 * 16], 128, 16),        # 1024 rows: the most that waves merge of so few splits
    (128, [516], [64 * 16], 128, 16),        # lanes, two rounds
    (64, [516], [64 * 9 - 3], 128, 9),       # a second round with one split
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


@pytest.mark.parametrize("call", ["gather", "sequence"])
@pytest.mark.parametrize("head_dim,n_q,n_doc", [(128, 130, 9000), (128, 37, 9000), (64, 300, 14000), (64, 41, 9000)])
def test_partials_of_the_other_calls(call, head_dim, n_q, n_doc):
    """Split rows of attention that reads the store and of a packed sequence: whole tiles, remainders and the rows of the last
    tile that do not exist.  Positions 0 and the bound as above."""
    from paper_2410_07590_amd import binding as B
    hq = 8
    gs = H.gpu_shape(B, synth.Shape(hq, 1, head_dim, "bf16", 1e4, 0))
    g = torch.Generator().manual_seed(head_dim + n_q)
    q = torch.randn(n_q, hq, head_dim, generator=g).bfloat16()
    k, v = (torch.randn(n_doc + n_q, 1, head_dim, generator=g).bfloat16() for _ in range(2))
    kd, vd = k.cuda(), v.cuda()
    if call == "gather":
        store = B.Store(gs, kd[:n_doc].contiguous(), vd[:n_doc].contiguous(), np.array([0, 4000, n_doc], np.int64))
        ids, off = np.array([0, 1], np.int32), np.array([0, 4000, n_doc], np.int64)
        out = torch.full_like(q, float("nan")).cuda()
        need = B.tr_prefill_attn_gather_workspace_size(store, ids, off, B.TR_POS_COMPOSITE, n_q)
        B.tr_prefill_attn_gather(store, ids, off, B.TR_POS_COMPOSITE, q.cuda(), kd, vd, torch.zeros(n_q, dtype=torch.int32).cuda(), out, B.workspace(need))
        rows_min = n_q * hq
    else:
        seg = np.concatenate([np.zeros(4000), np.full(n_doc - 4000, 4000), np.zeros(n_q)]).astype(np.int32)
        qs = torch.cat([torch.zeros(n_doc, hq, head_dim).bfloat16(), q]).cuda()
        full = torch.full_like(qs, float("nan"))
        need = B.tr_sequence_prefill_attn_workspace_size(gs, seg, n_doc + n_q)
        B.tr_sequence_prefill_attn(gs, qs, kd, vd, torch.from_numpy(seg).cuda(), torch.zeros(n_doc + n_q, dtype=torch.int32).cuda(), full,
                                   torch.empty_like(kd), seg_start_host=seg, workspace=B.workspace(need))
        assert not torch.isnan(full.float()).any()
        out = full[n_doc:]
        rows_min = n_q * hq
    assert need > 2 * rows_min * head_dim * 2     # split at all
    s = torch.matmul(q.double().reshape(n_q * hq, head_dim), k[:, 0].double().T) / head_dim ** 0.5
    hidden = torch.arange(n_doc + n_q)[None, :] > torch.arange(n_doc, n_doc + n_q).repeat_interleave(hq)[:, None]
    want = torch.matmul(torch.softmax(s.masked_fill(hidden, float("-inf")), 1), v[:, 0].double()).reshape(n_q, hq, head_dim)
    worst = ((out.cpu().double() - want).norm(dim=-1) / want.norm(dim=-1)).reshape(-1)
    assert not worst.isnan().any() and worst.max() < 1e-2, (int(worst.argmax()), float(worst.max()))
