"""Parity of the k-bit quantised convolution (sec. 3.2, "k-bit Quantization") with the CPU oracle, through the
C ABI: the int8 level numerators and the integer sum bit-exact, the scaled output within 1e-6 relative
(float(num) * float(1 / (La * Lw)) against the oracle's double quotient rounded once)."""
import numpy as np
import pytest
import torch

from oracle import xnor_oracle as xo
from paper_1603_05279_amd import xnor
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu

# n, c, h, w, k_out, kh, kw, stride, pad, ka, kw_bits
CASES = [
    (1, 1, 1, 1, 1, 1, 1, (1, 1), (0, 0), 1, 1),
    (2, 3, 5, 7, 2, 3, 3, (1, 1), (1, 1), 2, 1),
    (2, 33, 9, 8, 31, 3, 2, (1, 1), (1, 0), 2, 2),
    (3, 40, 11, 13, 70, 3, 3, (2, 2), (1, 1), 3, 1),
    (2, 17, 6, 6, 129, 1, 1, (1, 1), (0, 0), 4, 2),
    (5, 64, 14, 14, 64, 3, 3, (1, 1), (1, 1), 2, 2),
    (2, 96, 27, 27, 40, 5, 5, (1, 1), (2, 2), 1, 3),
    (1, 100, 7, 7, 20, 3, 3, (1, 1), (1, 1), 7, 7),
]


def run(x, W, stride, pad, ka, kb):
    n, c, h, w = x.shape
    k, _, kh, kw = W.shape
    desc = xnor.make_desc(n, c, h, w, k, kh, kw, stride, pad)
    ho, wo = xnor.output_hw(desc)
    dev = "cuda"
    xq = torch.full((xnor.kbit_input_bytes(n, c, h, w),), 99, dtype=torch.uint8, device=dev)
    wq = torch.empty((xnor.kbit_wimg_bytes(k, c, kh, kw),), dtype=torch.uint8, device=dev)
    scale = torch.zeros((k,), dtype=torch.float32, device=dev)
    out = torch.full((n, k, ho, wo), float("nan"), dtype=torch.float32, device=dev)
    num = torch.empty((n, k, ho, wo), dtype=torch.int32, device=dev)
    xnor.xnor_kbit_pack_weights(to_dev(W), scale, wq, ka, kb, k, c, kh, kw)
    xnor.xnor_kbit_pack_input(to_dev(x), xq, ka, n, c, h, w)
    xnor.xnor_kbit_conv2d(xq, wq, scale, out, num, desc, ka, kb)
    torch.cuda.synchronize()
    assert (scale.cpu().numpy() == np.float32(1.0 / (((1 << ka) - 1) * ((1 << kb) - 1)))).all()
    cw = (c + 31) // 32
    return out.cpu().numpy(), num.cpu().numpy(), xq.cpu().numpy().view(np.int8).reshape(n, h, w, cw * 32)


def levels_image(a):
    """numerators a = 2u - L [n][c][h][w] -> the packed tensor [n][h][w][cw*32] int8, 0 past the last channel"""
    n, c, h, w = a.shape
    cw = (c + 31) // 32
    img = np.zeros((n, h, w, cw * 32), dtype=np.int8)
    img[..., :c] = np.transpose(a, (0, 2, 3, 1)).astype(np.int8)
    return img


@pytest.mark.parametrize("case", CASES)
def test_kbit_conv_matches_oracle(case):
    n, c, h, w, k, kh, kw, stride, pad, ka, kb = case
    print("case", case, flush=True)
    rng = np.random.default_rng(11 + c + k)
    x = rng.uniform(-1.2, 1.2, (n, c, h, w)).astype(np.float32)          # some values beyond [-1, 1]: clamped
    W = rng.uniform(-1, 1, (k, c, kh, kw)).astype(np.float32)
    x.flat[:3] = [0.0, -0.0, 1.0]
    out, num, xq = run(x, W, stride, pad, ka, kb)
    r = xo.kbit_conv2d(x, W, ka, kb, stride, pad)
    assert np.array_equal(xq, levels_image(xo.qk_levels(x, ka)))
    assert np.array_equal(num.astype(np.int64), r["num"])
    np.testing.assert_allclose(out, r["out"], rtol=1e-6, atol=0)


def test_one_bit_each_is_the_binary_dot_map():
    rng = np.random.default_rng(2)
    x = rng.uniform(-1, 1, (2, 48, 9, 9)).astype(np.float32)
    W = rng.uniform(-1, 1, (24, 48, 3, 3)).astype(np.float32)
    out, num, _ = run(x, W, (1, 1), (1, 1), 1, 1)
    ref = xo.dot_map(xo.sign(x), xo.sign(W), (1, 1), (1, 1))
    assert np.array_equal(num, ref)
    assert np.array_equal(out, ref.astype(np.float32))


@pytest.mark.parametrize("k", range(1, 8))
def test_levels_of_special_values(k):
    # NaN, quiet or signaling, counts as -1; infinities, the ends of the range and their neighbours, denormal numbers, zeros of both signs
    words = [0x7F800001, 0xFF800001, 0x7FBFFFFF, 0x7FC00000, 0xFFC00001, 0x7F800000, 0xFF800000, 0x3F800000, 0x3F800001, 0x3F7FFFFF,
             0xBF800000, 0xBF800001, 0xBF7FFFFF, 0x80000000, 0, 1, 0x80000001, 0x33000000, 0xB3000000, 0x7F7FFFFF, 0xFF7FFFFF]
    x = np.resize(np.array(words, np.uint32), 64 * 40).view(np.float32).reshape(5, 64, 4, 2)
    xq = torch.full((xnor.kbit_input_bytes(*x.shape),), 99, dtype=torch.uint8, device="cuda")
    xnor.xnor_kbit_pack_input(to_dev(x), xq, k, *x.shape)
    assert np.array_equal(xq.cpu().numpy().view(np.int8).ravel(), levels_image(xo.qk_levels(x, k)).ravel())


def test_level_ties_and_errors():
    # inputs exactly halfway between two levels round up, like the oracle; NaN counts as -1
    k = 2
    x = np.array([0.0, -2.0 / 3.0, 2.0 / 3.0, np.nan, -1.0, 1.0, 1.0 / 3.0, -1.0 / 3.0], np.float32).reshape(1, 8, 1, 1)
    W = np.ones((1, 8, 1, 1), np.float32)
    out, num, xq = run(x, W, (1, 1), (0, 0), k, 1)
    assert np.array_equal(xq, levels_image(xo.qk_levels(x, k)))
    assert num.item() == int(xo.qk_levels(x, k).sum())
    with pytest.raises(xnor.XnorError) as e:
        xnor.xnor_kbit_pack_input(to_dev(x), torch.empty(32, dtype=torch.uint8, device="cuda"), 8, 1, 8, 1, 1)
    assert e.value.status == -2
    assert xnor.kbit_input_bytes(0, 8, 1, 1) == 0
    # 7 x 7 bits over 2^18 terms would overflow the 32-bit accumulator
    big = xnor.make_desc(1, 1 << 18, 1, 1, 1, 1, 1)
    z = torch.zeros(64, dtype=torch.uint8, device="cuda")
    with pytest.raises(xnor.XnorError) as e:
        xnor.xnor_kbit_conv2d(z, z, torch.zeros(4, device="cuda"), torch.zeros(4, device="cuda"), None, big, 7, 7)
    assert e.value.status == -3
