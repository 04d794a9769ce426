"""The extension module behind the binding: what it accepts, converts and refuses (CPU: nothing is enqueued)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2410_07590_amd import binding as B


@pytest.fixture(scope="module")
def store():
    B.lib()
    sh = B.make_shape(4, 4, 64, "f32", 1e4)
    sh_store = B.Store(sh, None, None, [0, 0, 0])  # two empty chunks: no memory is behind it
    return sh_store


@pytest.mark.parametrize("ids", [[1, 0, 1], (1, 0, 1), np.array([1, 0, 1], np.int64), np.array([1, 9, 0, 9, 1, 9], np.int32)[::2],
                                 np.array([1.0, 0.0, 1.0]), torch.tensor([1, 0, 1])])
def test_host_arrays_are_converted_as_numpy_does(store, ids):
    offsets, pos = B.tr_plan(store, ids, B.TR_POS_REORDERED)
    assert offsets.dtype == np.int64 and offsets.tolist() == [0, 0, 0, 0]
    assert pos.dtype == np.int32 and pos.size == 0
    assert B.tr_plan(store, ids, np.int32(0), want_pos_ids=False)[1] is None


def test_library_errors_and_wrong_arguments(store):
    with pytest.raises(B.TurboRagError) as e:
        B.tr_plan(store, [2], B.TR_POS_REORDERED)
    assert e.value.code == B.TR_ERR_BAD_CHUNK_ID and "chunk_ids[0]" in str(e.value)
    with pytest.raises(AssertionError):  # a host tensor where device memory is expected
        B.tr_kv_append(store.shape, torch.zeros(1, 4, 64), None, None, None, None, 0, stream=0)
    with pytest.raises(TypeError):
        B.tr_kv_append(store.shape, "k", None, None, None, None, 0, stream=0)
    with pytest.raises(AttributeError):
        B.tr_plan(None, [0], B.TR_POS_REORDERED)


def test_a_tensor_without_an_address_is_an_error_like_any_other():
    """A tensor that refuses its address (a traced one) makes the call raise.  In a process of its own: an exception that
    left the library call without the interpreter lock would end the process."""
    code = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2410_07590_amd import binding as B
with FakeTensorMode():
    x = torch.empty(2, 64, dtype=torch.bfloat16, device="cuda")
torch._C._set_throw_on_mutable_data_ptr(x)
try:
    B.tr_linear(x, [], [], stream=0)
except RuntimeError as e:
    print("refused:", "data pointer" in str(e))
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=root, timeout=300)
    assert res.returncode == 0 and "refused: True" in res.stdout, (res.returncode, res.stdout, res.stderr[-2000:])


def test_linear_takes_weights_with_trailing_dimensions():
    """A weight of shape [N, K, 1] (a convolution over one position) passes the shape check as it does with two dimensions:
    the call gets as far as the library, which refuses the missing memory of a tensor that has none."""
    from torch._subclasses.fake_tensor import FakeTensorMode
    with FakeTensorMode():
        x, y = (torch.empty(2, 64, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        good = [torch.empty(*s, dtype=torch.bfloat16, device="cuda") for s in ((64, 64), (64, 64, 1))]
        bad = [torch.empty(*s, dtype=torch.bfloat16, device="cuda") for s in ((64, 32), (64, 32, 2), (64,))]
    for w in good:
        with pytest.raises(B.TurboRagError, match="NULL pointer"):
            B.tr_linear(x, w, y, stream=0)
    for w in bad:
        with pytest.raises(AssertionError):
            B.tr_linear(x, w, y, stream=0)
