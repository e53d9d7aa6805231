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


# (the fused epilogue of 257 to 512 filters keeps up to 6 KiB of per-filter values and a word per pixel and 32 filters in LDS)
@pytest.mark.parametrize("case", [
    (15360, 64, 6, 6, 384, 6, 6, 1, 0), (6, 64, 8, 297, 384, 5, 5, 1, (3, 1)), (64, 7, 6, 700, 300, 5, 5, 2, 0), (39, 32, 54, 1076, 512, 3, 3, 2, 1),
    (2, 7, 16, 560, 256, 7, 7, 1, 0), (136, 64, 11, 301, 320, 5, 5, 1, 2)])
def test_fused_layers_with_wide_rows(case):
    d = ctypes.byref(xnor.make_desc(*case))
    for algo in (xnor.XNOR_ALGO_AUTO, xnor.XNOR_ALGO_MFMA_F4):
        assert xnor.lib().xnor_conv2d_binactiv(FAKE, FAKE, FAKE, None, FAKE, FAKE, None, None, FAKE, FAKE, None, FAKE, d, algo, None) == ERR_HIP


@pytest.mark.parametrize("case", [(2, 7, 8, 620, 300, 7, 7, 1, 1), (2, 64, 6, 400, 300, 5, 5, 1, 2), (168, 256, 14, 530, 256, 3, 3, (1, 2), 0)])
def test_plain_layers_with_wide_rows(case):
    d = ctypes.byref(xnor.make_desc(*case))
    for K, A in ((None, FAKE), (FAKE, None)):
        assert xnor.lib().xnor_conv2d(FAKE, FAKE, FAKE, K, A, FAKE, FAKE, None, d, xnor.XNOR_ALGO_MFMA_F4, None) == ERR_HIP


@pytest.mark.parametrize("case", [(7, 160, 6, 302, 256, 5, 7, 2, (2, 4)), (2, 352, 8, 213, 320, 7, 7, 1, 3), (300, 160, 8, 900, 256, 2, 2, 2, 0)])
def test_backward_layers_with_wide_rows(case):
    d = ctypes.byref(xnor.make_desc(*case))
    assert xnor.lib().xnor_bingrad_conv2d(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, d, xnor.XNOR_ALGO_MFMA_F4, None) == ERR_HIP


# (up to 16 channels: the parts are the faster form, and their image does not fit)
@pytest.mark.parametrize("case", [(1072, 8, 7, 8, 512, 7, 7, (1, 2), (6, 0)), (112, 10, 278, 72, 512, 3, 3, (4, 2), (2, 0)), (8, 5, 34, 85, 512, 7, 5, (2, 3), (2, 4))])
def test_binary_weight_layers_that_only_digits_stage(case):
    assert xnor.lib().xnor_bwn_conv2d(FAKE, FAKE, FAKE, FAKE, ctypes.byref(xnor.make_desc(*case)), None) == ERR_HIP


# Real inputs of more than 32 channels on rows so wide that the larger tiles' do not fit as digits (144 bytes a pixel and word) nor as parts
# (112): 129 to 640 filters, for which tiles of 64 to 96 pixels would, of many workgroups
@pytest.mark.parametrize("case", [
    (1, 64, 384, 384, 256, 3, 3, 2, 1), (32, 64, 384, 384, 256, 3, 3, 2, 1), (52, 96, 170, 176, 192, 3, 3, 2, 1),
    (75, 128, 53, 189, 192, 3, 3, 2, 1), (32, 96, 160, 160, 256, 5, 5, 2, 2), (128, 64, 192, 192, 256, 7, 7, 2, 3), (2, 64, 92, 92, 160, 7, 7, 1, 3),
    (4, 64, 184, 184, 160, 5, 5, 1, 2), (8, 48, 46, 92, 256, 7, 7, 1, 3), (1, 48, 98, 98, 640, 11, 11, 1, 5), (797, 35, 26, 345, 156, 1, 1, 3, 0),
    (2, 996, 93, 93, 2844, 7, 7, 2, (6, 3)), (301, 51, 36, 36, 441, 11, 1, 3, (5, 0)), (3, 34, 74, 160, 4278, 3, 7, 2, (0, 6))])
def test_binary_weight_layers_with_wide_rows(case):
    assert xnor.lib().xnor_bwn_conv2d(FAKE, FAKE, FAKE, FAKE, ctypes.byref(xnor.make_desc(*case)), None) == ERR_HIP


# (385 to 512 filters, up to 32 channels: 96 pixels do not fit as digits, 64 do)
@pytest.mark.parametrize("case", [(840, 25, 3, 23, 466, 5, 5, 3, (4, 3)), (207, 2, 36, 27, 433, 5, 7, 3, (0, 3))])
def test_binary_weight_layers_of_many_filters(case):
    assert xnor.lib().xnor_bwn_conv2d(FAKE, FAKE, FAKE, FAKE, ctypes.byref(xnor.make_desc(*case)), None) == ERR_HIP


# (sixteen waves leave room for 7680 channels, eight for 7936, four for 8064)
@pytest.mark.parametrize("n,c,h,w", [(1, 7681, 1, 2), (512, 7700, 2, 2), (1, 7936, 7, 7), (256, 7971, 13, 21), (512, 8000, 8, 8), (512, 8000, 2, 2), (3, 8064, 1, 3)])
def test_binactiv_up_to_the_channels_that_four_waves_hold(n, c, h, w):
    d = ctypes.byref(xnor.make_desc(n, c, h, w, 1, 1, 1))
    assert xnor.lib().xnor_binactiv(FAKE, None, None, FAKE, FAKE, None, d, None) == ERR_HIP
    assert xnor.lib().xnor_binarize_pack(FAKE, None, None, FAKE, n, c, h, w, None) == ERR_HIP
    assert xnor.lib().xnor_compute_K(FAKE, None, None, FAKE, FAKE, d, None) == ERR_HIP
