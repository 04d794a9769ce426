"""Attention of one token per request: contexts that end on either side of a unit of keys, and batches whose launch is cut in each
of the ways there are (one piece per request, about one piece per compute unit, many pieces), against a plain fp64 softmax."""
import numpy as np
import pytest
import torch

from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 159, 160, 161, 255, 256, 257, 288, 289, 383, 385, 511, 513, 640]


@pytest.mark.parametrize("hq,hkv,head_dim,lens,pieces", [
    (32, 8, 128, EDGES, "few"),                               # 208 (request, head) pairs
    (4, 4, 64, EDGES, "few"),
    (56, 8, 128, [300] * 64, "one"),                          # 512 pairs, none of them long
    (16, 8, 64, [200 + i for i in range(40)], "one"),
    (32, 8, 128, [6500] + [150 + 7 * i for i in range(24)], "many"),
    (8, 8, 64, [140 * i + 5 for i in range(40)], "many"),
    (2, 2, 128, [8191, 1], "few"),
])
def test_decode_pieces(hq, hkv, head_dim, lens, pieces):
    """1e-2 as for every bf16 attention (queries, weights and results in bf16 show 3e-3).  Positions are 0: nothing is rotated."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(hq, hkv, head_dim, "bf16", 1e4, 0)
    gs, g, n = H.gpu_shape(B, sh), hq // hkv, len(lens)
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    k, v = (torch.randn(int(start[-1]), hkv, head_dim, generator=gen, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn(n, hq, head_dim, generator=gen, device="cuda").bfloat16()
    need = B.tr_decode_attn_workspace_size(gs, start)
    most = n * hq * 64 * (head_dim * 2 + 8)                   # 64 pieces each
    assert need <= most and (need == 0) == (pieces == "one")
    if pieces == "many":
        assert need > 256 * g * (head_dim * 2 + 8)            # more than a piece per compute unit
    ws = B.workspace(need)
    ws.fill_(0xFF)                                            # partials that nobody writes would be NaN
    out = torch.full_like(q, float("nan"))
    B.tr_decode_attn(gs, q, k, v, torch.zeros(n, dtype=torch.int32, device="cuda"), start, out, ws)
    for r in range(n):
        kr, vr = (x[start[r]:start[r + 1]].double().cpu().repeat_interleave(g, 1) for x in (k, v))
        s = (kr * q[r].double().cpu()).sum(-1) / head_dim ** 0.5
        want = (torch.softmax(s, 0)[:, :, None] * vr).sum(0)
        err = (out[r].double().cpu() - want).norm(dim=-1) / want.norm(dim=-1)
        assert err.max() < 1e-2, (r, lens[r], float(err.max()))
