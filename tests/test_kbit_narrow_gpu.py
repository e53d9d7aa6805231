"""k-bit convolutions of at most two bits (4-bit operands) and their neighbours on int8, at the edges of words, K-steps and
channel chunks: the integer sum bit-exact against the oracle, also where the two forms border on each other."""
import numpy as np
import pytest
import torch

from oracle import xnor_oracle as xo
from paper_1603_05279_amd import xnor
from tests.helpers import to_dev
from tests.test_kbit_gpu import run

pytestmark = pytest.mark.gpu

# n, c, h, w, k_out, kh, kw, stride, pad
CASES = [
    (1, 31, 4, 5, 3, 1, 1, (1, 1), (0, 0)), (2, 32, 7, 7, 33, 3, 3, (1, 1), (1, 1)), (3, 65, 9, 6, 40, 3, 2, (2, 1), (1, 0)),
    (2, 96, 13, 13, 130, 3, 3, (1, 1), (1, 1)), (1, 140, 6, 6, 20, 3, 3, (1, 1), (1, 1)),      # five words: int8
    (2, 192, 11, 11, 257, 3, 3, (1, 1), (1, 1)), (1, 512, 40, 40, 32, 5, 5, (1, 1), (2, 2)),   # several chunks
    (1, 70, 5, 900, 130, 1, 1, (1, 1), (0, 0)), (2, 96, 16, 300, 3, 3, 3, (1, 1), (0, 0)),      # rows too wide for three words: int8
]


@pytest.mark.parametrize("bits", [(1, 1), (1, 2), (2, 1), (2, 2), (3, 2), (2, 3)])
@pytest.mark.parametrize("case", CASES)
def test_numerators_and_results(case, bits):
    n, c, h, w, k, kh, kw, stride, pad = case
    ka, kb = bits
    if c == 512 and bits != (2, 2):
        pytest.skip("one width of the largest case")
    print("case", case, bits, flush=True)
    rng = np.random.default_rng(c + 10 * ka + kb)
    x = rng.uniform(-1.1, 1.1, (n, c, h, w)).astype(np.float32)
    W = rng.uniform(-1.1, 1.1, (k, c, kh, kw)).astype(np.float32)
    out, num, _ = run(x, W, stride, pad, ka, kb)
    r = xo.kbit_conv2d(x, W, ka, kb, stride, pad)
    assert np.array_equal(num.astype(np.int64), r["num"])
    np.testing.assert_allclose(out, r["out"], rtol=1e-6, atol=0)


@pytest.mark.parametrize("kb,packed_ka", [(1, 1), (2, 2), (2, 5), (1, 7), (3, 2)])
def test_one_weight_image_serves_inputs_of_every_width(kb, packed_ka):
    # ka reaches the packer for `scale` alone: the same image under inputs of 1, 2 (4-bit operands) and 3, 7 bits (int8)
    n, c, h, k = 2, 65, 7, 40
    rng = np.random.default_rng(10 * kb + packed_ka)
    x = rng.uniform(-1.1, 1.1, (n, c, h, h)).astype(np.float32)
    W = rng.uniform(-1.1, 1.1, (k, c, 3, 3)).astype(np.float32)
    desc = xnor.make_desc(n, c, h, h, k, 3, 3, 1, 1)
    wq = torch.full((xnor.kbit_wimg_bytes(k, c, 3, 3),), 0x5A, dtype=torch.uint8, device="cuda")
    scale, out = torch.empty((k,), device="cuda"), torch.empty((n, k, h, h), device="cuda")
    num = torch.empty((n, k, h, h), dtype=torch.int32, device="cuda")
    xnor.xnor_kbit_pack_weights(to_dev(W), scale, wq, packed_ka, kb, k, c, 3, 3)
    for ka in (1, 2, 3, 7):
        xq = torch.empty((xnor.kbit_input_bytes(n, c, h, h),), dtype=torch.uint8, device="cuda")
        xnor.xnor_kbit_pack_input(to_dev(x), xq, ka, n, c, h, h)
        xnor.xnor_kbit_conv2d(xq, wq, scale, out, num, desc, ka, kb)
        r = xo.kbit_conv2d(x, W, ka, kb, (1, 1), (1, 1))
        assert np.array_equal(num.cpu().numpy().astype(np.int64), r["num"]), ka
