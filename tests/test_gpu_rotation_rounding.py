"""Rotated bf16 keys are rounded once from fp64, for every bf16 value a key can hold (subnormals, infinities and NaN among them) and
for results that a rounding by way of fp32 would get wrong, and angles are right up to the largest position id."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def append_at(B, sh, k, pos):
    ck, cv = torch.empty_like(k), torch.empty_like(k)
    B.tr_kv_append(H.gpu_shape(B, sh), k, k, torch.from_numpy(pos.astype(np.int32)).cuda(), ck, cv, 0)
    torch.cuda.synchronize()
    assert np.array_equal(H.bits_t(cv), H.bits_t(k))
    return H.bits(ck.cpu())


@pytest.mark.parametrize("kv_heads,head_dim,layout", [(4, 128, 0), (4, 128, 1), (2, 64, 0), (3, 64, 1)])
def test_every_value(kv_heads, head_dim, layout):
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(kv_heads, kv_heads, head_dim, "bf16", 1e4, layout)
    rng = np.random.Generator(np.random.PCG64([61, head_dim, layout]))
    row = kv_heads * head_dim
    rows = -(-4 * 65536 // row)
    k = np.concatenate([np.arange(65536), rng.permutation(65536), rng.integers(0, 256, 65536), np.arange(rows * row - 3 * 65536) % 65536])
    k = k.astype(np.uint16).reshape(rows, kv_heads, head_dim)   # whole range twice, subnormals of one sign, the range again
    pos = np.arange(rows) % 5 * 977
    with np.errstate(all="ignore"):
        want = oracle.rope(k, pos, sh.rope_base, layout)
    got = append_at(B, sh, torch.from_numpy(k.view(np.int16)).view(torch.bfloat16).cuda(), pos)
    nan = np.isnan(want)
    assert (got[nan] == 0x7fc0).all()
    H.assert_same_bits(got[~nan], oracle.round_to(want[~nan], oracle.BF16), "rotated keys", 1e-5)


@pytest.mark.parametrize("layout", [0, 1])
def test_every_position(layout):
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(1, 1, 128, "f32", 5e5, layout)
    rng = np.random.Generator(np.random.PCG64([62, layout]))
    pos = np.concatenate([np.arange(9), 2 ** np.arange(4, 31) - 1, 2 ** np.arange(4, 31), [2 ** 31 - 1], rng.integers(0, 2 ** 31, 60)])
    k = synth.normal_tensor(rng, (pos.size, 1, 128), torch.float32)
    got = append_at(B, sh, k.cuda(), pos)
    want = oracle.rope(H.bits(k), pos, sh.rope_base, layout)
    H.assert_same_bits(got, oracle.round_to(want, oracle.F32), "rotated keys", 1e-4)


@pytest.mark.parametrize("kv_heads,head_dim,layout", [(1, 128, 0), (1, 128, 1), (2, 64, 0), (3, 64, 1)])
def test_values_beside_a_tie(kv_heads, head_dim, layout):
    """Results whose fp32 rounding is a bf16 tie that they are not: rounded twice, about half of them would go to the wrong side.
    One in 2^16 is such a one; the rows that have them are picked out and their elements have to be right without exception."""
    from paper_2410_07590_amd import binding as B
    sh = synth.Shape(kv_heads, kv_heads, head_dim, "bf16", 1e4, layout)
    rng = np.random.Generator(np.random.PCG64([63, head_dim, layout]))
    rows = 20_000_000 // (kv_heads * head_dim)
    k = synth.as_oracle_array(synth.normal_tensor(rng, (rows, kv_heads, head_dim), torch.bfloat16))
    pos = rng.integers(1, 5000, rows)
    y = oracle.rope(k, pos, sh.rope_base, layout)
    y32 = y.astype(np.float32)
    tie = (y32.view(np.uint32) & 0xffff) == 0x8000
    # farther from the tie than sine and cosine of host and device can lie apart
    tie &= np.abs(y - y32) > 1e-15 * np.abs(oracle.widen(k)).max(axis=-1, keepdims=True)
    want = oracle.round_to(y, oracle.BF16)
    picked = tie.any(axis=(1, 2))
    tie, want, twice = tie[picked], want[picked], oracle.round_to(y32[picked].astype(np.float64), oracle.BF16)
    assert tie.sum() > 200 and (want[tie] != twice[tie]).sum() > 80
    got = append_at(B, sh, torch.from_numpy(k[picked].view(np.int16)).view(torch.bfloat16).cuda(), pos[picked])
    assert np.array_equal(got[tie], want[tie])
