"""fp32 attention at the edges of its key batches (4 keys for each group of lanes, four groups to a wave at head_dim 64, two at
128) with every number of waves per row that the rule chooses, against the oracle and fp64."""
import numpy as np
import pytest

from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,n_doc,n_q,layout", [
    (64, 1, 1, 0),        # two keys: all groups but two are empty
    (64, 125, 4, 1),      # eight waves, rows that see 126 .. 129 keys, the batch being 128
    (64, 253, 4, 1),      # 254 .. 257 keys: two batches
    (64, 600, 3, 0),      # a remainder in the fifth batch
    (128, 61, 5, 0),      # 62 .. 66 keys, the batch being 64
    (128, 125, 5, 0),
    (128, 300, 2, 1),
    (64, 380, 130, 1),    # 520 rows: four waves per row, 381 .. 510 keys in batches of 64
    (128, 125, 130, 0),   # 126 .. 255 keys
    (64, 61, 1030, 0),    # 4 x 1030 rows of 62 .. 1091 keys: four waves
    (64, 1000, 300, 0),   # 1200 rows of about as many keys
    (128, 1000, 300, 1),
    (128, 30, 513, 1),    # 2052 rows: four waves, batches of 32
    (128, 5, 3, 0),       # two waves
    (128, 5, 1, 0),       # one
])
def test_f32_attention_edges(head_dim, n_doc, n_q, layout):
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(4, 2, head_dim, "f32", 1e4, layout)
    rng = np.random.Generator(np.random.PCG64([31, head_dim, n_doc, n_q]))
    row_start = np.array([0, n_doc], np.int64)

    def draw(n, heads):
        return synth.normal_tensor(rng, (n, heads, head_dim), sh.torch_dtype)

    store = synth.Store(draw(n_doc, 2), draw(n_doc, 2), row_start)
    sd = B.Store(H.gpu_shape(B, sh), store.k.cuda(), store.v.cuda(), row_start)
    req = synth.Request(np.array([0], np.int32), synth.POS_REORDERED, n_q, draw(n_q, 4), draw(n_q, 2), draw(n_q, 2),
                        (n_doc + np.arange(n_q)).astype(np.int32), n_doc, [n_doc])
    rows = None if n_q < 100 else np.linspace(0, n_q - 1, 40).astype(int)
    H.check_request(B, sh, store, sd, req, rows=rows, k_mismatch_frac=1e-4)


@pytest.mark.parametrize("head_dim,n_req,n_q,lo,hi", [
    (64, 40, 16, 1, 50),     # 2560 rows of 2 .. 65 keys: two waves per row, batches of 32
    (128, 40, 16, 1, 50),    # batches of 16
    (64, 9, 16, 1, 70),      # 576 rows: four waves, some of them without keys
    (64, 400, 16, 1, 30),    # 25600 rows: one wave
    (128, 400, 16, 1, 10),
    (128, 3, 5, 1, 20),      # 60 rows of few keys
])
def test_f32_rows_of_few_keys(head_dim, n_req, n_q, lo, hi):
    """Many requests over short caches, some keys with a score of -inf: every fourth (all the keys of one group of lanes) and a
    few more.  Positions are 0, so the result is a plain softmax, taken in fp64.  Error bound: fp32 sums of at most 70 values
    of size up to 5, 5 * 70 * 2^-24 < 3e-5."""
    import torch
    from paper_2410_07590_amd import binding as B
    gs = H.gpu_shape(B, synth.Shape(4, 2, head_dim, "f32", 1e4, 0))
    rng = np.random.Generator(np.random.PCG64([32, head_dim, n_req]))
    start = np.concatenate([[0], np.cumsum(rng.integers(lo, hi, n_req) + n_q)]).astype(np.int64)
    cu = (np.arange(n_req + 1) * n_q).astype(np.int32)
    g = torch.Generator().manual_seed(head_dim + n_req)
    q = torch.randn(n_req * n_q, 4, head_dim, generator=g).abs()     # times a key of -3e38 in every channel: -inf
    k, v = (torch.randn(int(start[-1]), 2, head_dim, generator=g) for _ in range(2))
    gone = torch.zeros(int(start[-1]), dtype=torch.bool)
    for r in range(n_req):
        gone[int(start[r]) + 1:int(start[r + 1]):4] = True
        gone[int(start[r]) + 6:int(start[r + 1]):16] = True
    k[gone] = -3e38
    out = torch.full_like(q, float("nan")).cuda()
    B.tr_prefill_attn_batched(gs, q.cuda(), k.cuda(), v.cuda(), torch.zeros(n_req * n_q, dtype=torch.int32).cuda(), cu, start, out,
                              B.workspace(B.tr_prefill_attn_batched_workspace_size(gs, cu, start)))
    out = out.cpu().double()
    for r in range(n_req):
        keys = slice(int(start[r]), int(start[r + 1]))
        n = keys.stop - keys.start
        s = torch.einsum("thd,khd->thk", q[cu[r]:cu[r + 1]].double(), k[keys].repeat_interleave(2, 1).double()) / head_dim ** 0.5
        hidden = torch.arange(n)[None, :] > torch.arange(n - n_q, n)[:, None]
        s = s.masked_fill((hidden | gone[keys][None])[:, None], float("-inf"))
        want = torch.einsum("thk,khd->thd", torch.softmax(s, -1), v[keys].repeat_interleave(2, 1).double())
        assert (out[cu[r]:cu[r + 1]] - want).abs().max() < 3e-5, r


@pytest.mark.parametrize("head_dim,n_q", [(64, 2), (64, 1030), (128, 2)])
def test_f32_attention_scores_that_overflow(head_dim, n_q):
    """Keys whose scores are -inf have weight 0, also where they are all the keys of one group of lanes' batch (every
    32nd, 16th, 8th or 4th key): with equal scores elsewhere the result is the mean over the other visible keys.  Error
    bound: fp32 sums of at most 1091 values of size 1, under 1e-5 relative to them."""
    import torch
    from paper_2410_07590_amd import binding as B
    n_doc = 61
    kv_len = n_doc + n_q
    gs = H.gpu_shape(B, synth.Shape(4, 2, head_dim, "f32", 1e4, 0))
    k = torch.zeros(kv_len, 2, head_dim)
    gone = torch.zeros(kv_len, dtype=torch.bool)
    gone[5::32] = True
    gone[3::16] = True
    gone[2::8] = True
    k[gone] = -3e38                                     # times a query of ones: the sum over the channels overflows
    v = torch.randn(kv_len, 2, head_dim, generator=torch.Generator().manual_seed(3))
    q = torch.ones(n_q, 4, head_dim)
    out = torch.empty_like(q).cuda()
    B.tr_prefill_attn(gs, q.cuda(), k.cuda(), v.cuda(), torch.zeros(n_q, dtype=torch.int32).cuda(), kv_len, out,
                      B.workspace(B.tr_prefill_attn_workspace_size(gs, n_q, kv_len)))
    w = (~gone).double()[:, None, None]
    mean = (torch.cumsum(v.double() * w, 0) / torch.cumsum(w, 0))[n_doc:]
    want = mean.repeat_interleave(2, 1)
    assert (out.cpu().double() - want).abs().max() < 1e-5
