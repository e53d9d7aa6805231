"""Geometries near the limits of the LDS plans: the matrix-core launchers have to take them.  Without a device a call that
passes every check and every plan ends with the HIP error of its launch; one that is refused gives XNOR_ERR_UNSUPPORTED."""
import ctypes

import pytest
import torch

from paper_1603_05279_amd import xnor

ERR_HIP = -5
FAKE = ctypes.c_void_p(0x1000)          # never dereferenced: there is no device to launch on

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="would launch on the fake pointers")


# n, c, h, w, k_out, kh, kw, stride, pad: three channel words and rows that do not fit with all three of them
@pytest.mark.parametrize("case", [
    (1, 70, 5, 900, 130, 1, 1, 1, 0), (1, 96, 10, 900, 1, 1, 1, 1, 0), (16, 96, 224, 224, 64, 7, 7, 2, 3), (1, 96, 400, 400, 64, 5, 5, 1, 2),
    (8, 96, 320, 320, 128, 3, 3, 2, 1), (2, 96, 480, 640, 128, 3, 3, 1, 1), (4, 96, 300, 300, 64, 5, 5, 1, 2)])
def test_kbit_layers_of_two_bits_are_taken_where_three_bits_are(case):
    d = ctypes.byref(xnor.make_desc(*case))
    for ka, kb in ((1, 1), (1, 2), (2, 2), (2, 3), (3, 3)):
        assert xnor.lib().xnor_kbit_conv2d(FAKE, FAKE, FAKE, FAKE, None, d, ka, kb, None) == ERR_HIP
