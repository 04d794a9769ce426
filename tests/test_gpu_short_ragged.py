"""Batches of short queries over contexts of very different lengths: their launch is cut into many pieces only to even it out, and
what the pieces hold must lose nothing against one workgroup per request and head.  Values far from one (bf16 has fp32's range),
several query tokens with their causal edge at and beside the ends of pieces, rotated queries in both layouts; against fp64."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

LONG = [6500] + [150 + 7 * i for i in range(24)]            # 200 (request, head) pairs of 8 heads
RISING = [140 * i + 5 for i in range(40)]                   # 320 pairs
EDGES = [256 * i + e for i in (1, 4, 9, 16) for e in (-2, -1, 0, 1, 2, 3, 4, 127, 128, 129)] + [20, 5]   # query tokens on both sides of a piece's end


def inputs(sh, lens, n_q, scale, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    k, v = (torch.randn(int(start[-1]), sh.n_kv_heads, sh.head_dim, generator=gen, device="cuda") for _ in range(2))
    q = torch.randn(n_q * len(lens), sh.n_q_heads, sh.head_dim, generator=gen, device="cuda").bfloat16()
    pos = np.repeat(np.array(lens) - n_q, n_q) + np.tile(np.arange(n_q), len(lens)) + 31
    cu = (n_q * np.arange(len(lens) + 1)).astype(np.int32)
    return q, k.bfloat16(), (v * scale).bfloat16(), pos, cu, start


def attend(B, sh, q, k, v, pos, cu, start, ws):
    out = torch.full_like(q, float("nan"))
    B.tr_prefill_attn_batched(H.gpu_shape(B, sh), q, k, v, torch.from_numpy(pos.astype(np.int32)).cuda(), cu, start, out, ws)
    torch.cuda.synchronize()
    return out


def worst_error(sh, out, q, k, v, pos, cu, start):
    """Largest relative error of an output row against fp64."""
    g, worst = sh.n_q_heads // sh.n_kv_heads, 0.0
    turned = torch.from_numpy(oracle.rope(H.bits(q.cpu()), pos, sh.rope_base, sh.rope_layout)).cuda().double()
    for r in range(len(cu) - 1):
        toks, n_q, n = slice(int(cu[r]), int(cu[r + 1])), int(cu[r + 1] - cu[r]), int(start[r + 1] - start[r])
        hidden = torch.arange(n, device="cuda")[None, :] > torch.arange(n - n_q, n, device="cuda").repeat_interleave(g)[:, None]
        for h in range(sh.n_kv_heads):
            heads = slice(h * g, (h + 1) * g)
            keys, vals = (x[int(start[r]):int(start[r + 1]), h].double().contiguous() for x in (k, v))
            s = turned[toks, heads].reshape(n_q * g, -1) @ keys.t().contiguous() / sh.head_dim ** 0.5
            want = torch.softmax(s.masked_fill(hidden, float("-inf")), 1) @ vals
            got = out[toks, heads].double().reshape(n_q * g, -1)
            err = float(((got - want).norm(dim=1) / want.norm(dim=1)).max())
            assert err == err, "request %d, head %d: not finite" % (r, h)
            worst = max(worst, err)
    return worst


@pytest.mark.parametrize("hq,hkv,head_dim,layout,lens,n_q,scale", [
    (32, 8, 128, 0, LONG, 1, 1.0),
    (32, 8, 128, 1, LONG, 1, 1e-6),
    (32, 8, 128, 0, RISING, 1, 1e-6),
    (8, 8, 64, 1, RISING, 1, 1e5),
    (16, 8, 64, 0, RISING, 4, 1e-7),
    (16, 8, 128, 1, EDGES, 4, 1.0),
    (32, 8, 64, 1, EDGES, 5, 1e5),
    (56, 8, 128, 0, EDGES, 3, 1e-5),
])
def test_many_pieces(hq, hkv, head_dim, layout, lens, n_q, scale):
    """1e-2 as for every bf16 attention (queries, weights and results in bf16 show 3e-3): no operation in it depends on the scale of
    the values, so the bound does not either."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(hq, hkv, head_dim, "bf16", 1e4, layout)
    lens = [max(n, n_q) for n in lens]
    q, k, v, pos, cu, start = inputs(sh, lens, n_q, scale, len(lens) + n_q)
    need = B.tr_prefill_attn_batched_workspace_size(H.gpu_shape(B, sh), cu, start)
    assert need > 256 * n_q * (hq // hkv) * (head_dim * 2 + 8)     # more than a piece per compute unit
    ws = B.workspace(need)
    ws.fill_(0xFF)                                                 # partials that nobody writes would be NaN
    err = worst_error(sh, attend(B, sh, q, k, v, pos, cu, start, ws), q, k, v, pos, cu, start)
    print("%d requests, %d tokens, values of %g: %.2e" % (len(lens), n_q, scale, err))
    assert err < 1e-2


@pytest.mark.parametrize("layout,lens,n_q", [(0, RISING, 1), (1, RISING, 4), (0, LONG, 1)])
def test_less_workspace(layout, lens, n_q):
    """Without room for the many pieces a batch runs with the cut that fills the chip, which is none from 256 pairs on; less room than
    that is refused, and nothing is written."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(32, 8, 128, "bf16", 1e4, layout)
    lens = [max(n, n_q) for n in lens]
    q, k, v, pos, cu, start = inputs(sh, lens, n_q, 1.0, len(lens) + n_q)
    need = B.tr_prefill_attn_batched_workspace_size(H.gpu_shape(B, sh), cu, start)
    rows = 0 if len(lens) * 8 >= 256 else 2 * n_q * 32 * sum(n > 256 for n in lens)   # two pieces each, of requests that can be cut
    least = -(-rows * 256 // 256) * 256 + -(-rows * 8 // 256) * 256
    assert least < need - 256
    room = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    for ws in [room, room[:need - 256], room[:least]] + ([room[:0], None] if least == 0 else []):
        room.fill_(0xFF)
        err = worst_error(sh, attend(B, sh, q, k, v, pos, cu, start, ws), q, k, v, pos, cu, start)
        assert err < 1e-2, (None if ws is None else ws.numel(), err)
        assert ws is None or bool((room[ws.numel():] == 0xFF).all())
    for ws in [room[:least - 256], room[16:], None] if least else []:
        with pytest.raises(B.TurboRagError) as e:
            attend(B, sh, q, k, v, pos, cu, start, ws)
        assert e.value.code == B.TR_ERR_WORKSPACE


@pytest.mark.parametrize("layout,lens", [(0, RISING), (1, LONG)])
def test_rows_without_weight(layout, lens):
    """A row all of whose scores are minus infinity is zero, whether its request is cut or not; a piece without weight changes
    nothing for the others."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(8, 8, 128, "bf16", 1e4, layout)
    q, k, v, pos, cu, start = inputs(sh, lens, 1, 1.0, 77)
    pos[:] = 0
    q[:, :, 0] = 1.0
    need = B.tr_decode_attn_workspace_size(H.gpu_shape(B, sh), start)
    last = slice(int(start[-2]), int(start[-1]))     # one request without any weight
    k[last, :, 0] = float("-inf")
    first = slice(int(start[0]), int(start[0]) + max(1, lens[0] - 300)) if lens[0] > 600 else slice(int(start[-3]), int(start[-3]) + 4000)
    k[first, :, 0] = float("-inf")                   # and one whose first pieces have none
    out = attend(B, sh, q, k, v, pos, cu, start, B.workspace(need))
    assert bool((out[-1] == 0).all())
    if lens is RISING:
        assert bool((attend(B, sh, q, k, v, pos, cu, start, None)[-1] == 0).all())   # the same batch, uncut
    k[last, :, 0] = 0.0
    assert worst_error(sh, out[:-1], q[:-1], k, v, pos[:-1], cu[:-1], start[:-1]) < 1e-2


def test_static_array_holds_the_many_pieces():
    """One request whose pairs leave CUs idle (96 heads of up to 256 CUs, 24 MB of partials): the library's own array, same bits."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(96, 96, 128, "bf16", 1e4, 0)
    q, k, v, pos, cu, start = inputs(sh, [8192], 32, 1e-6, 5)
    need = B.tr_prefill_attn_workspace_size(H.gpu_shape(B, sh), 32, 8192)
    assert 256 * 32 * (128 * 2 + 8) < need <= B.tr_prefill_attn_static_scratch_bytes()
    want = attend(B, sh, q, k, v, pos, cu, start, B.workspace(need))
    assert worst_error(sh, want, q, k, v, pos, cu, start) < 1e-2
    got = torch.full_like(q, float("nan"))
    B.tr_prefill_attn_static(H.gpu_shape(B, sh), q, k, v, torch.from_numpy(pos.astype(np.int32)).cuda(), 8192, got)
    torch.cuda.synchronize()
    assert torch.equal(H.bits_t(got), H.bits_t(want))
