"""What GatedConv.forward_beside hands to the library, without a GPU: the call itself is replaced by one that notes its arguments."""
from types import SimpleNamespace

import pytest
import torch

from paper_1805_12549_amd import binding as B


@pytest.fixture
def call(monkeypatch):
    seen = []
    monkeypatch.setattr(B._lib, "cg_conv_call_beside", lambda *args: seen.append(args) or B.CG_OK)
    layer = object.__new__(B.GatedConv)
    layer.handle, layer.stream, layer.ho, layer.wo, layer.c_out = None, SimpleNamespace(cuda_stream=0), 4, 3, 128
    layer._y_dtype, layer.desc = torch.bfloat16, SimpleNamespace(c_in=64)
    return layer, seen


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_outputs_are_of_their_layers_type(call, dtype):
    """(float outputs went into a tensor of bf16)"""
    layer, seen = call
    layer._y_dtype = dtype
    x, w1, one = torch.zeros((2, 4, 3, 64), dtype=torch.bfloat16), torch.zeros((192, 64), dtype=torch.bfloat16), torch.ones(192)
    y, y1 = layer.forward_beside(x, w1, one, None, 192)
    assert (y.dtype, y.shape, y.is_contiguous()) == (dtype, (2, 4, 3, 128), True)
    assert (y1.dtype, y1.shape, y1.is_contiguous()) == (torch.bfloat16, (2, 4, 3, 192), True)
    assert seen == [(None, 2, x.data_ptr(), y.data_ptr(), w1.data_ptr(), one.data_ptr(), 0, y1.data_ptr(), 192, 0, 0)]


@pytest.mark.parametrize("w1,scale,shift", [((128, 64), 192, 192), ((192, 32), 192, 192), ((192, 64), 128, 192), ((192, 64), None, 191), ((256, 64), 192, 192)])
def test_a_1x1_of_other_sizes_is_refused(call, w1, scale, shift):
    """(its operands were read as far as the number of channels said)"""
    layer, seen = call
    with pytest.raises(B.CGError):
        layer.forward_beside(torch.zeros((2, 4, 3, 64), dtype=torch.bfloat16), torch.zeros(w1, dtype=torch.bfloat16), None if scale is None else torch.ones(scale),
                             torch.ones(shift), 192)
    assert seen == []
