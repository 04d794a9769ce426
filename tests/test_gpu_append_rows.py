"""Appended cache rows at the edges of the kernel's walk: rows shorter and longer than what a group of lanes owns (128 units of
16 bytes at 128 channels, 64 at 64, where a wave has two groups), tokens that do not fill a workgroup, and numbers of requests
around one and two rounds of the run search (64) and around what one launch carries (128); and launches of so many short rows
that tokens share a group.  Whole numbers are
compared: the oracle rotates in fp64 and rounds once."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_kv,head_dim,dtype,layout,n_req,longest,empty", [
    (1, 64, "bf16", 0, 1, 1, 0),       # 8 units: most of the wave idle
    (1, 64, "bf16", 1, 9, 1, 0),       # two tokens to a wave, of two requests
    (8, 64, "bf16", 0, 70, 2, 5),      # 64 units: a full group
    (9, 64, "bf16", 1, 5, 3, 0),       # 72 units: two groups, a wave to a token
    (17, 64, "bf16", 1, 67, 2, 0),     # 136 units: three groups, so that tokens share waves and cross them
    (13, 64, "f32", 0, 66, 2, 7),      # 208 units: four groups
    (4, 128, "bf16", 1, 1, 7, 0),      # 64 units, tokens not a multiple of a workgroup's four
    (8, 128, "bf16", 0, 64, 1, 0),     # one round of the search, full
    (3, 64, "bf16", 1, 65, 3, 0),      # a second round with one entry
    (3, 64, "bf16", 1, 65, 3, 30),     # and requests of no tokens among them
    (8, 128, "bf16", 1, 128, 2, 0),    # all that a launch carries
    (2, 128, "bf16", 0, 129, 2, 0),    # two launches, one request in the second
    (2, 128, "bf16", 0, 131, 2, 40),
    (8, 64, "f32", 1, 259, 1, 0),      # three launches
    (17, 128, "bf16", 1, 3, 9, 0),     # 272 units: a third group with a remainder
    (40, 128, "f32", 0, 2, 5, 0),      # 1280 units: ten whole groups
    (9, 128, "f32", 1, 66, 2, 3),      # 288 units
    (5, 64, "f32", 0, 5, 4, 1),
])
def test_appended_rows(n_kv, head_dim, dtype, layout, n_req, longest, empty):
    """n_req requests with tokens, which is what the launch counts, and `empty` ones without at random places among them."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(n_kv, n_kv, head_dim, dtype, 5e5, layout)
    rng = np.random.Generator(np.random.PCG64([77, n_kv, head_dim, n_req]))
    n_q = np.concatenate([rng.integers(1, longest + 1, n_req - 1), [longest], np.zeros(empty, np.int64)])
    n_q = rng.permutation(n_q)
    assert (n_q > 0).sum() == n_req
    n_req += empty
    free = rng.integers(0, 3, n_req)                    # rows in front of the query tokens
    start = np.concatenate([[0], np.cumsum(n_q + free)]).astype(np.int64)
    cu = np.concatenate([[0], np.cumsum(n_q)]).astype(np.int32)
    total, rows = int(cu[-1]), int(start[-1])
    k = synth.normal_tensor(rng, (total, n_kv, head_dim), sh.torch_dtype)
    v = synth.normal_tensor(rng, (total, n_kv, head_dim), sh.torch_dtype)
    pos = rng.integers(0, 40000, total).astype(np.int32)
    ck = torch.full((rows + 2, n_kv, head_dim), float("nan"), dtype=sh.torch_dtype, device="cuda")
    cv = torch.full_like(ck, float("nan"))
    B.tr_kv_append_batched(H.gpu_shape(B, sh), k.cuda(), v.cuda(), torch.from_numpy(pos).cuda(), cu, start, ck, cv)
    torch.cuda.synchronize()
    dst = np.concatenate([np.arange(start[r + 1] - n_q[r], start[r + 1]) for r in range(n_req)]).astype(np.int64)
    want = oracle.round_to(oracle.rope(H.bits(k), pos, sh.rope_base, layout), oracle.F32 if dtype == "f32" else oracle.BF16)
    # fp32 results round 29 bits of the fp64 value instead of 45: a last-bit difference of the two libraries' sincos shows
    # once in about 2^28 values; the few thousand here see none, and a share of 1e-4 would be noticed
    H.assert_same_bits(H.bits(ck.cpu())[dst], want, "appended keys", 1e-4 if dtype == "f32" else 1e-5)
    H.assert_same_bits(H.bits(cv.cpu())[dst], H.bits(v), "appended values")
    rest = np.setdiff1d(np.arange(rows + 2), dst)
    assert torch.isnan(ck.cpu().float()[rest]).all() and torch.isnan(cv.cpu().float()[rest]).all()


@pytest.mark.parametrize("n_kv,head_dim,dtype,layout,n_req,total,by", [
    (1, 64, "bf16", 0, 1, 8192, 0),      # the fewest tokens that share a group: eight to a wave
    (1, 64, "bf16", 1, 70, 8195, 1),     # runs that begin inside a wave, a last wave that is not full, rows at odd elements
    (2, 64, "bf16", 0, 90, 16384, 3),    # two heads per lane
    (2, 64, "bf16", 1, 128, 16389, 0),
    (1, 128, "bf16", 0, 2, 4099, 0),     # four to a wave
    (2, 128, "bf16", 1, 3, 8195, 0),
    (1, 64, "f32", 1, 1, 8193, 1),
    (1, 64, "f32", 0, 40, 8192, 0),
    (3, 64, "bf16", 0, 90, 20001, 3),    # more than half of the lanes busy: a group to a token, many of them
])
def test_many_short_rows(n_kv, head_dim, dtype, layout, n_req, total, by):
    """Launches in which tokens share a group give the bits that launches of few tokens give, a group to a token."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(n_kv, n_kv, head_dim, dtype, 5e5, layout)
    gs = H.gpu_shape(B, sh)
    rng = np.random.Generator(np.random.PCG64([78, n_kv, head_dim, total]))
    cut = np.sort(rng.choice(total - 1, n_req - 1, replace=False) + 1)
    cu = np.concatenate([[0], cut, [total]]).astype(np.int32)     # every request has a token
    start = cu.astype(np.int64) + np.arange(n_req + 1)            # and a row in front of them
    rows, pos = int(start[-1]), torch.from_numpy(rng.integers(0, 40000, total).astype(np.int32)).cuda()

    def view(n, value=None):     # `by` elements into its allocation
        room = torch.full((n * n_kv * head_dim + 8,), float("nan"), dtype=sh.torch_dtype, device="cuda")
        t = room[by:by + n * n_kv * head_dim].view(n, n_kv, head_dim)
        return t if value is None else t.copy_(value)

    k, v = (view(total, synth.normal_tensor(rng, (total, n_kv, head_dim), sh.torch_dtype)) for _ in range(2))
    ck, cv = view(rows), view(rows)
    B.tr_kv_append_batched(gs, k, v, pos, cu, start, ck, cv)
    want_k, want_v = torch.empty_like(k), torch.empty_like(v)
    for t0 in range(0, total, 1000):
        t1 = min(t0 + 1000, total)
        B.tr_kv_append(gs, k[t0:t1], v[t0:t1], pos[t0:t1], want_k[t0:t1], want_v[t0:t1], 0)
    dst = torch.from_numpy(np.concatenate([np.arange(start[r] + 1, start[r + 1]) for r in range(n_req)])).cuda()
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(ck[dst].view(bits), want_k.view(bits)) and torch.equal(cv[dst].view(bits), want_v.view(bits))
    assert torch.equal(cv[dst], v)
    rest = torch.from_numpy(start[:-1]).cuda()
    assert torch.isnan(ck[rest].float()).all() and torch.isnan(cv[rest].float()).all()


@pytest.mark.parametrize("dtype,layout,n_q", [("bf16", 0, 1), ("bf16", 1, 6), ("f32", 0, 3), ("f32", 1, 2)])
def test_rows_that_start_at_any_element(dtype, layout, n_q):
    """Views whose first element is not 16-byte aligned: the appended rows have the bits that aligned copies give."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(3, 3, 64, dtype, 1e4, layout)
    gs = H.gpu_shape(B, sh)
    g = torch.Generator().manual_seed(9)

    def off(t, by):     # a copy that starts `by` elements into its allocation
        room = torch.zeros(t.numel() + 16, dtype=t.dtype, device="cuda")
        room[by:by + t.numel()] = t.reshape(-1).cuda()
        return room[by:by + t.numel()].view(t.shape)

    k, v = (torch.randn(n_q, 3, 64, generator=g).to(sh.torch_dtype) for _ in range(2))
    pos = torch.arange(7, 7 + n_q, dtype=torch.int32).cuda()
    got = {}
    for by in (0, 1, 3):
        ck, cv = off(torch.zeros_like(k), by), off(torch.zeros_like(v), by)
        B.tr_kv_append(gs, off(k, by), off(v, by), pos, ck, cv, 0)
        got[by] = (ck.cpu().clone(), cv.cpu().clone())
    for by in (1, 3):
        assert torch.equal(got[by][0], got[0][0]) and torch.equal(got[by][1], got[0][1]) and torch.equal(got[by][1], v)


@pytest.mark.parametrize("n_kv,head_dim,dtype,layout", [(1, 64, "bf16", 0), (17, 64, "bf16", 1), (3, 64, "f32", 1), (9, 128, "bf16", 0), (40, 128, "f32", 1)])
@pytest.mark.parametrize("n_q", [1, 6, 27])
def test_rows_appended_by_the_launch_that_assembles(n_kv, head_dim, dtype, layout, n_q):
    """Bytes of the two calls, for rows of one to ten groups of lanes, and nothing behind the last token."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(n_kv, n_kv, head_dim, dtype, 5e5, layout)
    gs = H.gpu_shape(B, sh)
    rng = np.random.Generator(np.random.PCG64([79, n_kv, head_dim, n_q]))
    rows = np.array([0, 5, 40], np.int64)
    ks, vs = (synth.normal_tensor(rng, (40, n_kv, head_dim), sh.torch_dtype).cuda() for _ in range(2))
    store = B.Store(gs, ks, vs, rows)
    ids = np.array([1, 0], np.int32)
    offsets, _ = B.tr_plan(store, ids, B.TR_POS_REORDERED, want_pos_ids=False)
    k, v = (synth.normal_tensor(rng, (n_q, n_kv, head_dim), sh.torch_dtype).cuda() for _ in range(2))
    pos = torch.arange(40, 40 + n_q, dtype=torch.int32, device="cuda")
    got, want = (torch.full((2, 40 + n_q + 3, n_kv, head_dim), float("nan"), dtype=sh.torch_dtype, device="cuda") for _ in range(2))
    B.tr_kv_assemble_append(store, ids, offsets, B.TR_POS_REORDERED, k, v, pos, got[0], got[1])
    B.tr_kv_assemble(store, ids, offsets, B.TR_POS_REORDERED, want[0], want[1])
    B.tr_kv_append(gs, k, v, pos, want[0], want[1], 40)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(got.view(bits), want.view(bits))
    assert not torch.isnan(got[:, :40 + n_q].float()).any()
