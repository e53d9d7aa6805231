"""k-bit convolutions of at most two bits (4-bit operands) and their neighbours on int8, at the edges of words, K-steps and
channel chunks: the integer sum bit-exact against the oracle, also where the two forms border on each other."""
import numpy as np
import pytest

from oracle import xnor_oracle as xo
from tests.test_kbit_gpu import run

pytestmark = pytest.mark.gpu

# n, c, h, w, k_out, kh, kw, stride, pad
CASES = [
    (1, 31, 4, 5, 3, 1, 1, (1, 1), (0, 0)), (2, 32, 7, 7, 33, 3, 3, (1, 1), (1, 1)), (3, 65, 9, 6, 40, 3, 2, (2, 1), (1, 0)),
    (2, 96, 13, 13, 130, 3, 3, (1, 1), (1, 1)), (1, 140, 6, 6, 20, 3, 3, (1, 1), (1, 1)),      # five words: int8
    (2, 192, 11, 11, 257, 3, 3, (1, 1), (1, 1)), (1, 512, 40, 40, 32, 5, 5, (1, 1), (2, 2)),   # several chunks
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
