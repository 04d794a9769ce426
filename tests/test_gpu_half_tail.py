"""Walks whose last 64-key tile holds at most 32 keys, and their neighbours: one key, a half tile, a key more, a whole tile;
alone, after whole tiles, in both ring depths, for packed chunks and for queries behind a document prefix."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture
def B():
    from paper_2410_07590_amd import binding
    yield binding
    binding.tr_set_tuning("wg_rows", 0)


def _draw(rng, sh, n, heads):
    return synth.normal_tensor(rng, (n, heads, sh.head_dim), sh.torch_dtype)


SHAPES = [synth.LLAMA3_8B, synth.Shape(14, 2, 64, "bf16", 1e6, 1), synth.Shape(4, 4, 128, "bf16", 1e4, 1)]


@pytest.mark.parametrize("wg_rows", [128, 256])
@pytest.mark.parametrize("sh", SHAPES, ids=lambda s: "%dx%d" % (s.n_q_heads, s.head_dim))
def test_packed_chunks(B, sh, wg_rows):
    """Chunks one token to five tiles long, so that row tiles end at every remainder and also straddle chunks."""
    B.tr_set_tuning("wg_rows", wg_rows)
    cu = np.concatenate([[0], np.cumsum((32, 1, 31, 33, 64, 65, 96, 97, 63, 160, 161, 300, 2))]).astype(np.int32)
    T = int(cu[-1])
    rng = np.random.Generator(np.random.PCG64([91, sh.head_dim, wg_rows]))
    q, k, v = _draw(rng, sh, T, sh.n_q_heads), _draw(rng, sh, T, sh.n_kv_heads), _draw(rng, sh, T, sh.n_kv_heads)
    gs = H.gpu_shape(B, sh)
    out, k_rot = torch.full_like(q, float("nan"), device="cuda"), torch.empty_like(k, device="cuda")
    ws = B.workspace(B.tr_chunk_prefill_attn_workspace_size(gs, T, 300))
    B.tr_chunk_prefill_attn(gs, q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(cu).cuda(), cu.size - 1, 300, out, k_rot, ws)
    torch.cuda.synchronize()
    want = oracle.offline_chunk_prefill(H.bits(q), H.bits(k), H.bits(v), cu, sh.rope_base, layout=sh.rope_layout)["out"]
    assert float(np.abs(H.to_f64(out.cpu()) - want).max()) <= H.tol_for(sh)


@pytest.mark.parametrize("wg_rows", [128, 256])
@pytest.mark.parametrize("sh", SHAPES, ids=lambda s: "%dx%d" % (s.n_q_heads, s.head_dim))
@pytest.mark.parametrize("n_doc,n_q", [(1, 5), (26, 5), (27, 5), (28, 6), (59, 5), (60, 5), (91, 5), (92, 5), (291, 29), (300, 90), (700, 37)])
def test_queries_behind_documents(B, sh, n_doc, n_q, wg_rows):
    """Requests of n_doc + n_q keys: 6 to 737, the remainder below, at and above a half tile."""
    B.tr_set_tuning("wg_rows", wg_rows)
    rng = np.random.Generator(np.random.PCG64([92, sh.head_dim, n_doc, n_q]))
    row_start = np.array([0, n_doc], np.int64)
    store = synth.Store(_draw(rng, sh, n_doc, sh.n_kv_heads), _draw(rng, sh, n_doc, sh.n_kv_heads), row_start)
    sd = B.Store(H.gpu_shape(B, sh), store.k.cuda(), store.v.cuda(), row_start)
    req = synth.Request(np.array([0], np.int32), synth.POS_REORDERED, n_q, _draw(rng, sh, n_q, sh.n_q_heads),
                        _draw(rng, sh, n_q, sh.n_kv_heads), _draw(rng, sh, n_q, sh.n_kv_heads), (n_doc + np.arange(n_q)).astype(np.int32), n_doc, [n_doc])
    H.check_request(B, sh, store, sd, req, k_mismatch_frac=1e-4)
