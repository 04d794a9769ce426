"""Keys rotated by the offline call with angles from its table (many tokens) and with angles of the rotation kernel's own (few):
the same fp64 arithmetic, so the same bits for the tokens that a short and a long call share."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

LINE = 12288 * 64   # angles up to which a call has no table (interleaved pairs: counting half a workgroup of the rotation kernel
                    # more for each chunk); the test sees which side it is on by what the call writes


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("kv_heads,head_dim", [(1, 128), (9, 64), (2, 64)])
def test_both_sides_of_the_line(dtype, layout, kv_heads, head_dim):
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(kv_heads, kv_heads, head_dim, dtype, 1e6, layout)
    gs = H.gpu_shape(B, sh)
    extra = 0 if layout else 2048 // (head_dim * (2 if dtype == "bf16" else 4))
    room = lambda lens: LINE // (head_dim // 2) - sum(lens) - extra * (len(lens) + 1)   # for one more chunk
    lens = [1, 700, 33, 64]
    while room(lens) > 160:
        lens.append(128)
    lens.append(room(lens))
    edge, T = sum(lens), sum(lens) + 1
    rng = np.random.Generator(np.random.PCG64([93, kv_heads, head_dim, layout]))
    q, k, v = (synth.normal_tensor(rng, (T, kv_heads, head_dim), sh.torch_dtype) for _ in range(3))

    def run(lens):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        n = int(cu[-1])
        out, k_rot = torch.empty_like(q[:n], device="cuda"), torch.empty_like(k[:n], device="cuda")
        ws = B.workspace(B.tr_chunk_prefill_attn_workspace_size(gs, n, 700))
        ws.fill_(0x5A)
        B.tr_chunk_prefill_attn(gs, q[:n].cuda(), k[:n].cuda(), v[:n].cuda(), torch.from_numpy(cu).cuda(), cu.size - 1, 700, out, k_rot, ws)
        torch.cuda.synchronize()
        table = ws[:700 * (head_dim // 2) * 16]      # the workspace starts with it: cosine and sine in fp64, position by pair
        return H.bits(k_rot.cpu()), H.bits(out.cpu()), not bool((table == 0x5A).all())

    k_own, out_own, has_table = run(lens)
    assert not has_table
    k_table, out_table, has_table = run(lens + [1])
    assert has_table
    assert np.array_equal(k_own, k_table[:edge]) and np.array_equal(out_own, out_table[:edge])
    few = 1 + 700 + 33
    cu = np.array([0, 1, 701, few], np.int32)
    want = oracle.offline_chunk_prefill(H.bits(q[:few]), H.bits(k[:few]), H.bits(v[:few]), cu, sh.rope_base, layout=layout, rows=np.array([0], np.int32))
    H.assert_same_bits(k_own[:few], want["k_rot_st"], "rotated keys K'", 1e-5)
