"""The weight packer's images byte for byte, at the edges of its work split: 8-filter groups, 32-channel words, runs of
at most 16 taps (one run up to 16 taps, several beyond), and filters, channels and blocks that end inside a record."""
import numpy as np
import pytest
import torch

from paper_1603_05279_amd import xnor
from tests.helpers import pack_signs_channels_last, to_dev

pytestmark = pytest.mark.gpu

# k_out, c, kh, kw
CASES = [(1, 1, 1, 1), (7, 31, 1, 1), (8, 33, 1, 1), (9, 520, 1, 1), (33, 32, 3, 3), (5, 3, 11, 11), (31, 65, 4, 4),
         (10, 31, 1, 17), (64, 96, 5, 5), (3, 40, 64, 64)]


def padded_signs(W):
    """sign(W) as [filter blocks * 32][taps][Cw * 32], 0 past the last filter and channel."""
    k, c, kh, kw = W.shape
    s = np.zeros(((k + 31) // 32 * 32, kh * kw, (c + 31) // 32 * 32), dtype=np.int8)
    s[:k, :, :c] = np.where(W >= 0, 1, -1).reshape(k, c, kh * kw).transpose(0, 2, 1)
    return s


def expected_images(W):
    s = padded_signs(W)
    fb, taps, cw = s.shape[0] // 32, s.shape[1], s.shape[2] // 32
    zero = np.zeros(1024, dtype=np.uint8)
    # int8 records [block][tap][word]: half-wave, filter, 16 channels
    i8 = s.reshape(fb, 32, taps, cw, 2, 16).transpose(0, 2, 3, 4, 1, 5).reshape(-1).view(np.uint8)
    # 4-bit records: two (tap, word) blocks each, 32 filters x 32 channels of nibbles per block
    code = np.where(s > 0, 0x2, np.where(s < 0, 0xA, 0)).astype(np.uint8)
    nib = code.reshape(fb, 32, taps * cw, 32).transpose(0, 2, 1, 3)
    nib = (nib[..., 0::2] | nib[..., 1::2] << 4).reshape(fb, taps * cw, 512)
    if taps * cw % 2:
        nib = np.concatenate([nib, np.zeros((fb, 1, 512), np.uint8)], 1)
    words = np.packbits((s > 0).reshape(fb, 32, taps * cw, 32), axis=-1, bitorder="little")
    words = words.reshape(fb, 32, taps * cw, 4).transpose(0, 2, 1, 3).reshape(-1)
    return np.concatenate([i8, zero, nib.reshape(-1), zero, words])


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("transposed", [False, True])
def test_weight_images(case, transposed):
    k, c, kh, kw = case
    print("case", case, transposed, flush=True)
    rng = np.random.default_rng(k * 1000 + c)
    W = rng.standard_normal((k, c, kh, kw)).astype(np.float32)
    W.reshape(-1)[::5] = 0.0
    W.reshape(-1)[::7] *= -0.0                                   # -0.0 counts as +1
    F = np.ascontiguousarray(W[:, :, ::-1, ::-1].transpose(1, 0, 2, 3)) if transposed else W   # the filters packed
    fk, fc = F.shape[:2]
    guard = 64
    nbytes = xnor.wmfma_bytes(fk, fc, kh, kw)
    img = torch.full((nbytes + guard,), 0x5A, dtype=torch.uint8, device="cuda")
    bits = torch.full((fk, kh * kw, (fc + 31) // 32), -1, dtype=torch.int32, device="cuda")
    factor = torch.full((fk,), -1.0, device="cuda")
    if transposed:
        xnor.xnor_bingrad_pack_weights(to_dev(W), bits, factor, img, k, c, kh, kw)
    else:
        xnor.xnor_pack_weights(to_dev(W), bits, factor, img, k, c, kh, kw)
    got = img.cpu().numpy()
    assert np.array_equal(got[:nbytes], expected_images(F))
    assert (got[nbytes:] == 0x5A).all()
    signs = np.where(F >= 0, 1, -1).astype(np.int32)
    assert np.array_equal(bits.cpu().numpy().view(np.uint32),
                          pack_signs_channels_last(signs).reshape(fk, kh * kw, (fc + 31) // 32))
    expect = np.ones(fk) if transposed else np.abs(F.astype(np.float64)).mean((1, 2, 3))
    # a float sum of n terms of one sign: at most n / 256 + 9 roundings on any path of the tree
    assert np.allclose(factor.cpu().numpy(), expect, rtol=(F[0].size / 256 + 10) * 2.0 ** -24, atol=0)


def test_more_groups_than_workgroups():
    # one filter value each: k_out / 8 image groups and k_out alpha groups, past the 2^22 workgroups of a launch by less
    # than a turn (the first ones take a second turn)
    k = (1 << 22) - (1 << 18)
    rng = np.random.default_rng(22)
    W = rng.standard_normal((k, 1, 1, 1)).astype(np.float32)
    bits = torch.full((k, 1, 1), -1, dtype=torch.int32, device="cuda")
    factor = torch.full((k,), -1.0, device="cuda")
    xnor.xnor_pack_weights(to_dev(W), bits, factor, None, k, 1, 1, 1)
    assert k + k // 8 > 1 << 22
    assert np.array_equal(bits.cpu().numpy().reshape(-1), (W.reshape(-1) >= 0).astype(np.int32))
    assert np.array_equal(factor.cpu().numpy(), np.abs(W.reshape(-1)))
