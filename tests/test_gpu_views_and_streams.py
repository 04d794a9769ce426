"""Arguments that a caller may pass in more than one form: tensors that begin at any element of their allocation where the
kernels' wide accesses are declared for that, and the stream as torch's current one, as an object or as a raw handle."""
import numpy as np
import pytest
import torch

from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def at(t, by):
    """A copy of t on the GPU that begins `by` elements into its allocation (which is aligned to 256 bytes)."""
    room = torch.zeros(t.numel() + 16, dtype=t.dtype, device="cuda")
    return room[by:by + t.numel()].view(t.shape).copy_(t)


def empty_at(shape, dtype, by):
    return at(torch.full(shape, float("nan"), dtype=dtype, device="cuda"), by)


def randn(*size, seed, dtype=torch.bfloat16):
    return torch.randn(size, generator=torch.Generator().manual_seed(seed)).to(dtype).cuda()


def same_for_every_start(call, shape, dtype):
    """call(by, out) fills out; the bits are those of an output that begins on a 256-byte boundary."""
    want = empty_at(shape, dtype, 0)
    call(0, want)
    assert not torch.isnan(want.float()).any()
    for by in (1, 3, 6):
        got = empty_at(shape, dtype, by)
        call(by, got)
        assert np.array_equal(H.bits_t(got), H.bits_t(want)), "output from element %d on" % by


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads,n_q,kv_len,split", [
    ((4, 2), 40, 60, False),      # rows straight from the attention kernel's registers
    ((4, 2), 40, 3000, True),     # from the merge, a few lanes per row
    ((2, 1), 20, 6000, True),     # from the merge, a wave per row
    ((8, 1), 300, 700, False),
])
def test_prefill_output_at_any_element(head_dim, heads, n_q, kv_len, split):
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(*heads, head_dim, "bf16", 1e4, 0))
    q = randn(n_q, heads[0], head_dim, seed=1)
    k, v = (randn(kv_len, heads[1], head_dim, seed=s) for s in (2, 3))
    pos = torch.arange(kv_len - n_q, kv_len, dtype=torch.int32, device="cuda")
    B.tr_set_tuning("wg_rows", 128)
    B.tr_set_tuning("target_items", 0 if split else 1)
    try:
        need = B.tr_prefill_attn_workspace_size(gs, n_q, kv_len)
        assert (need > 0) == split
        same_for_every_start(lambda by, out: B.tr_prefill_attn(gs, q, k, v, pos, kv_len, out, B.workspace(need)), q.shape, q.dtype)
    finally:
        B.tr_set_tuning("wg_rows", 0)
        B.tr_set_tuning("target_items", 0)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("lens", [[100, 20, 300], [5000, 77]])
def test_decode_output_at_any_element(head_dim, lens):
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(4, 2, head_dim, "bf16", 1e4, 0))
    start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    q = randn(len(lens), 4, head_dim, seed=4)
    k, v = (randn(int(start[-1]), 2, head_dim, seed=s) for s in (5, 6))
    pos = torch.tensor(lens, dtype=torch.int32).cuda() - 1
    ws = B.workspace(B.tr_decode_attn_workspace_size(gs, start))
    same_for_every_start(lambda by, out: B.tr_decode_attn(gs, q, k, v, pos, start, out, ws), q.shape, q.dtype)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_other_outputs_at_any_element(head_dim):
    """Attention that reads the store, packed chunks, and a packed sequence whose last tokens walk everything (split keys)."""
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(4, 2, head_dim, "bf16", 1e4, 1))
    lens, n_q = [70, 200, 33], 17
    rows, n_doc = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), sum(lens)
    k, v = (randn(n_doc, 2, head_dim, seed=s) for s in (7, 8))
    store = B.Store(gs, k, v, rows)
    ids = np.array([2, 0, 1], np.int32)
    offsets, _ = B.tr_plan(store, ids, B.TR_POS_REORDERED, want_pos_ids=False)
    q = randn(n_q, 4, head_dim, seed=9)
    ck, cv = (randn(n_doc + n_q, 2, head_dim, seed=s) for s in (10, 11))
    pos = torch.arange(n_doc, n_doc + n_q, dtype=torch.int32, device="cuda")
    ws = B.workspace(B.tr_prefill_attn_gather_workspace_size(store, ids, offsets, B.TR_POS_REORDERED, n_q))
    same_for_every_start(lambda by, out: B.tr_prefill_attn_gather(store, ids, offsets, B.TR_POS_REORDERED, q, ck, cv, pos, out, ws), q.shape, q.dtype)

    cu = torch.from_numpy(rows.astype(np.int32)).cuda()
    qd = randn(n_doc, 4, head_dim, seed=12)
    ws2 = B.workspace(B.tr_chunk_prefill_attn_workspace_size(gs, n_doc, max(lens)))
    rot = torch.empty_like(k)
    same_for_every_start(lambda by, out: B.tr_chunk_prefill_attn(gs, qd, k, v, cu, 3, max(lens), out, rot, ws2), qd.shape, qd.dtype)

    seg, sp = B.tr_sequence_plan(np.full(40, 128, np.int32), 30, B.TR_POS_COMPOSITE)
    t = len(seg)
    qs, ks, vs = randn(t, 4, head_dim, seed=13), randn(t, 2, head_dim, seed=14), randn(t, 2, head_dim, seed=15)
    seg_d, sp_d, rot2 = torch.from_numpy(seg).cuda(), torch.from_numpy(sp).cuda(), torch.empty_like(ks)
    need = B.tr_sequence_prefill_attn_workspace_size(gs, seg, t)
    assert need > 0
    ws3 = B.workspace(need)
    same_for_every_start(lambda by, out: B.tr_sequence_prefill_attn(gs, qs, ks, vs, seg_d, sp_d, out, rot2, seg_start_host=seg, workspace=ws3),
                         qs.shape, qs.dtype)


@pytest.mark.parametrize("head_dim,n_q,kv_len", [(64, 5, 40), (128, 130, 300)])
def test_fp32_attention_at_any_element(head_dim, n_q, kv_len):
    """Queries, keys and values too."""
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(4, 2, head_dim, "f32", 1e4, 0))
    q = randn(n_q, 4, head_dim, seed=16, dtype=torch.float32)
    k, v = (randn(kv_len, 2, head_dim, seed=s, dtype=torch.float32) for s in (17, 18))
    pos = torch.arange(kv_len - n_q, kv_len, dtype=torch.int32, device="cuda")
    same_for_every_start(lambda by, out: B.tr_prefill_attn(gs, at(q, by), at(k, by), at(v, by), pos, kv_len, out), q.shape, q.dtype)


@pytest.mark.parametrize("form", ["current", "object", "handle", "default"])
def test_calls_are_enqueued_on_the_stream_that_was_asked_for(form):
    """The inputs reach their buffers on a side stream, behind a wait of some milliseconds: a call enqueued anywhere else
    would not see them.  "default": with the side stream current, an explicit handle of 0 is the default stream all the same."""
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(4, 2, 128, "bf16", 1e4, 0))
    n, kv_len = 9, 50
    q, k, v = randn(n, 4, 128, seed=20), randn(n, 2, 128, seed=21), randn(n, 2, 128, seed=22)
    ck, cv = randn(kv_len, 2, 128, seed=23), randn(kv_len, 2, 128, seed=24)
    pos = torch.arange(kv_len - n, kv_len, dtype=torch.int32, device="cuda")
    ws = B.workspace(B.tr_prefill_attn_workspace_size(gs, n, kv_len))

    def run(qx, kx, vx, stream):
        ckx, cvx, out = ck.clone(), cv.clone(), torch.full_like(q, float("nan"))
        torch.cuda.synchronize()
        return ckx, cvx, out, lambda: (B.tr_kv_append(gs, kx, vx, pos, ckx, cvx, kv_len - n, stream=stream),
                                       B.tr_prefill_attn(gs, qx, ckx, cvx, pos, kv_len, out, ws, stream=stream))

    want_k, want_v, want, go = run(q, k, v, None)
    go()
    zeros = run(torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v), None)
    zeros[3]()
    torch.cuda.synchronize()
    assert not torch.equal(zeros[2], want)

    side = torch.cuda.Stream()
    late = [torch.zeros_like(x) for x in (q, k, v)]
    asked = {"current": None, "object": side, "handle": side.cuda_stream, "default": 0}[form]
    got_k, got_v, got, go = run(*late, asked)
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        for x, y in zip(late, (q, k, v)):
            x.copy_(y)
        if form in ("current", "default"):
            go()
    if form in ("object", "handle"):
        go()
    torch.cuda.synchronize()
    expect = (want_k, want_v, want) if form != "default" else zeros[:3]
    for g, w in zip((got_k, got_v, got), expect):
        assert np.array_equal(H.bits_t(g), H.bits_t(w))
