"""The key-splitting kernel of very short queries, forced onto several row tiles: an early tile's causal end lies in front of the
second key split, so the workgroup of that pair walks no keys.  What it merges must not depend on the keys of later tokens, which
it requested all the same: here those keys are not finite."""
import numpy as np
import pytest
import torch

from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("hq,hkv,head_dim,n_doc,n_q,tiles_per_split", [
    (32, 8, 128, 230, 40, None),     # the second split starts at key 256: tiles 0 .. 2 (tokens 0 .. 23) end before it
    (32, 8, 64, 230, 40, None),
    (8, 1, 128, 120, 140, 1),        # three splits of 128 keys, 35 tiles
    (2, 2, 64, 5, 300, 1),           # one head per group: 32 tokens per tile, tiles that walk none of two splits
])
def test_rows_in_front_of_a_split(hq, hkv, head_dim, n_doc, n_q, tiles_per_split, bad):
    """Positions are 0, so the result is a plain softmax over the visible keys, taken in fp64; 1e-2 as for every bf16 attention
    (queries, weights and results in bf16 show 3e-3)."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(hq, hkv, head_dim, "bf16", 1e4, 0)
    gs, g, kv_len = H.gpu_shape(B, sh), hq // hkv, n_doc + n_q
    gen = torch.Generator().manual_seed(head_dim + n_q)
    q = torch.randn(n_q, hq, head_dim, generator=gen).bfloat16()
    k, v = (torch.randn(kv_len, hkv, head_dim, generator=gen).bfloat16() for _ in range(2))
    first_bad = kv_len - kv_len // 10                    # key of the first token whose own row is not finite
    n_good = first_bad - n_doc                           # tokens that see finite keys only
    kd = k.clone()
    kd[first_bad:, :, 1::2] = bad
    names = {"wg_rows": 32}
    if tiles_per_split:
        names.update(min_split_keys=128, target_items=4096)
    for name, value in names.items():
        B.tr_set_tuning(name, value)
    try:
        need = B.tr_prefill_attn_workspace_size(gs, n_q, kv_len)
        out = torch.full_like(q, float("nan")).cuda()
        ws = B.workspace(need)
        ws.fill_(0xFF)                                   # partials that nobody writes would be NaN
        assert need >= 2 * n_q * hq * head_dim * 2       # at least two splits
        B.tr_prefill_attn(gs, q.cuda(), kd.cuda(), v.cuda(), torch.zeros(n_q, dtype=torch.int32).cuda(), kv_len, out, ws)
        torch.cuda.synchronize()
    finally:
        for name in names:
            B.tr_set_tuning(name, 0)
    out = out.cpu().double()[:n_good]
    assert n_good > 0 and torch.isfinite(out).all()
    for h in range(hkv):
        s = torch.matmul(q[:n_good, h * g:(h + 1) * g].double().reshape(n_good * g, head_dim), k[:, h].double().T) / head_dim ** 0.5
        hidden = torch.arange(kv_len)[None, :] > torch.arange(n_doc, n_doc + n_good).repeat_interleave(g)[:, None]
        want = torch.matmul(torch.softmax(s.masked_fill(hidden, float("-inf")), 1), v[:, h].double()).reshape(n_good, g, head_dim)
        err = (out[:, h * g:(h + 1) * g] - want).norm(dim=-1) / want.norm(dim=-1)
        assert err.max() < 1e-2, (h, float(err.max()))
