"""Cache rows are stored in one of two ways, by how many bytes the call forms: calls on both sides of the line give the rows that
the store holds (bit for bit under composite positions) and the oracle's rotation of them (under reordered ones)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

THROUGH_MIN = 96 << 20   # bytes of K and V


@pytest.mark.parametrize("dtype,layout,kv_heads,head_dim,by", [
    ("bf16", 0, 4, 128, 0), ("bf16", 1, 4, 128, 1), ("f32", 0, 3, 64, 3), ("f32", 1, 3, 64, 0),
])
@pytest.mark.parametrize("formed", [THROUGH_MIN - 1, THROUGH_MIN])
def test_both_sides_of_the_line(dtype, layout, kv_heads, head_dim, by, formed):
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(kv_heads, kv_heads, head_dim, dtype, 1e6, layout)
    row_bytes = 2 * kv_heads * head_dim * (2 if dtype == "bf16" else 4)
    rows = formed // row_bytes if formed < THROUGH_MIN else -(-formed // row_bytes)
    assert (rows * row_bytes >= THROUGH_MIN) == (formed >= THROUGH_MIN) and abs(rows * row_bytes - THROUGH_MIN) <= row_bytes
    lens = [1, 333, 1024, 47, 700]
    ids = []
    while rows - sum(lens[i] for i in ids) > 1024:
        ids.append(len(ids) % len(lens))
    lens.append(rows - sum(lens[i] for i in ids))   # the last chunk is what is left
    ids = np.array(ids + [len(lens) - 1], np.int32)
    row_start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    g = torch.Generator().manual_seed(5)
    k, v = (torch.randn(int(row_start[-1]), kv_heads, head_dim, generator=g).to(sh.torch_dtype) for _ in range(2))
    store = B.Store(H.gpu_shape(B, sh), k.cuda(), v.cuda(), row_start)
    src = torch.cat([torch.arange(row_start[i], row_start[i + 1]) for i in ids]).cuda()
    room = torch.zeros(2, rows * kv_heads * head_dim + 16, dtype=sh.torch_dtype, device="cuda")
    ck, cv = (r[by:by + rows * kv_heads * head_dim].view(rows, kv_heads, head_dim) for r in room)
    for mode in (B.TR_POS_COMPOSITE, B.TR_POS_REORDERED):
        room.fill_(float("nan"))
        offsets, _ = B.tr_plan(store, ids, mode, want_pos_ids=False)
        B.tr_kv_assemble(store, ids, offsets, mode, ck, cv)
        torch.cuda.synchronize()
        assert torch.equal(cv, v.cuda()[src])
        assert bool(room[:, :by].isnan().all()) and bool(room[:, by + rows * kv_heads * head_dim:].isnan().all())
        if mode == B.TR_POS_COMPOSITE:
            assert torch.equal(ck, k.cuda()[src])
            continue
        assert not bool(ck.isnan().any())
        for j in (0, 2, len(ids) - 1):   # chunks at both ends and one of 1024 rows
            a, b = int(offsets[j]), int(offsets[j + 1])
            part = k[row_start[ids[j]]:row_start[ids[j] + 1]]
            want = oracle.rope(H.bits(part), np.full(b - a, a, np.int64), sh.rope_base, layout)
            H.assert_same_bits(H.bits(ck[a:b].cpu()), oracle.round_to(want, oracle._dtype_of(H.bits(part))), "rotated keys", 1e-4)
