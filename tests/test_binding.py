"""Argument checks of the binding (csrc/binding.cpp): what is refused before any entry point runs (no GPU)."""
import ctypes

import pytest
import torch

from paper_1603_05279_amd import xnor


def test_tensor_arguments_are_checked_before_the_call():
    d = xnor.make_desc(1, 64, 14, 14, 64, 3, 3, 1, 1)
    with pytest.raises(ValueError, match="device tensors"):
        xnor.xnor_binactiv(torch.zeros(4), None, None, None, None, None, d)
    with pytest.raises(TypeError):
        xnor.xnor_binactiv(3, None, None, None, None, None, d)
    with pytest.raises(TypeError):
        xnor.xnor_binactiv(None, None, None, None, None, None, 5)
    with pytest.raises(TypeError):
        xnor.xnor_binarize_pack(None, None, None, None, 1.5, 1, 1, 1)


class _OtherStructure(ctypes.Structure):
    _fields_ = [("v", ctypes.c_int * (ctypes.sizeof(xnor.ConvDesc) // 4))]


@pytest.mark.parametrize("other", [bytes(ctypes.sizeof(xnor.ConvDesc)), bytearray(ctypes.sizeof(xnor.ConvDesc)), _OtherStructure(),
                                   torch.zeros(ctypes.sizeof(xnor.ConvDesc), dtype=torch.uint8).numpy(), None])
def test_only_a_descriptor_is_a_descriptor(other):
    with pytest.raises(TypeError, match="descriptor"):
        xnor.xnor_binactiv(None, None, None, None, None, None, other, stream=_Stream())


class _Stream:
    cuda_stream = 0


def test_status_of_the_library_becomes_its_error():
    with pytest.raises(xnor.XnorError) as e:            # refused by the C ABI before it touches a device
        xnor.xnor_linear(None, None, None, None, None, None, None, 1, 1, 1, stream=_Stream())
    assert e.value.status == -1 and "xnor_linear" in str(e.value)


@pytest.mark.gpu
def test_device_tensors_of_another_type_or_layout():
    d = xnor.make_desc(1, 64, 14, 14, 64, 3, 3, 1, 1)
    x = torch.zeros((1, 64, 14, 14), device="cuda")
    with pytest.raises(ValueError, match="[Ff]loat"):
        xnor.xnor_binactiv(x.half(), None, None, None, None, None, d)
    with pytest.raises(ValueError, match="densely"):
        xnor.xnor_binactiv(x.transpose(2, 3)[:, :, 1:], None, None, None, None, None, d)
