"""Binary-Weight-Network convolution with its inputs as digits (filters of 25 taps and more take that form at any size) at the
edges of its words, K-steps and chunks, and with inputs at the ends of the float range.

A result is a float sum of c*kh*kw terms, each input held to half a unit in the last place of the largest of its 32-channel
word: |out - ref| <= alpha * (terms * 2^-24 * max |x| + 1e-5 * |ref|/alpha) covers both with room for the order of the sum."""
import numpy as np
import pytest
import torch

from oracle import xnor_oracle as xo
from tests.test_bwn_gpu import run

pytestmark = pytest.mark.gpu


def check(x, w, stride, pad):
    out, alpha, _ = run(x, w, stride, pad)
    ref = xo.bwn_conv2d(x, w, stride, pad)
    np.testing.assert_allclose(alpha, ref["alpha"], rtol=1e-5, atol=0)
    terms = w[0].size
    bound = ref["alpha"][None, :, None, None] * terms * 2.0 ** -24 * np.abs(x).max() + 1e-5 * np.abs(ref["out"])
    err = np.abs(out.astype(np.float64) - ref["out"])
    assert (err <= bound).all(), float((err / bound).max())
    return out


# n, c, h, w, k_out, kh, kw, stride, pad
CASES = [
    (1, 1, 5, 5, 1, 5, 5, (1, 1), (0, 0)), (2, 15, 7, 9, 33, 5, 5, (1, 1), (2, 2)), (2, 17, 9, 6, 70, 5, 5, (2, 1), (2, 2)),
    (3, 33, 8, 8, 130, 5, 5, (1, 1), (2, 2)), (2, 65, 13, 13, 257, 5, 5, (1, 1), (2, 2)), (1, 96, 27, 27, 64, 5, 5, (1, 1), (2, 2)),
    (2, 160, 14, 14, 100, 5, 5, (2, 2), (1, 2)), (1, 290, 20, 20, 40, 5, 7, (1, 1), (2, 3)), (1, 512, 9, 9, 512, 5, 5, (1, 1), (2, 2)),
    (40, 64, 24, 24, 128, 3, 3, (1, 1), (1, 1)),                 # 3 x 3 with workgroups enough for digits
    (8, 5, 34, 85, 512, 7, 5, (2, 3), (2, 4)),                   # parts are faster and do not fit
]


@pytest.mark.parametrize("case", CASES)
def test_matches_oracle(case):
    n, c, h, w, k, kh, kw, stride, pad = case
    print("case", case, flush=True)
    rng = np.random.default_rng(c * 100 + h)
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    x.flat[::11] = 0.0
    check(x, rng.standard_normal((k, c, kh, kw)).astype(np.float32), stride, pad)


@pytest.mark.parametrize("scale", [2.0 ** 100, 2.0 ** -90, 2.0 ** -108])
def test_magnitudes(scale):
    rng = np.random.default_rng(7)
    x = (rng.standard_normal((1, 48, 9, 9)) * scale).astype(np.float32)
    x[:, ::3] *= np.float32(2.0 ** -12)                          # small inputs beside large ones in every word
    w = (np.where(rng.standard_normal((20, 48, 5, 5)) >= 0, 1.0, -1.0)).astype(np.float32)
    check(x, w, (1, 1), (2, 2))


def test_sums_that_cancel_are_those_of_the_exact_inputs():
    # one word, inputs with 24-bit significands near one power of two: every digit sum is exact
    rng = np.random.default_rng(8)
    x = (1.0 + rng.integers(0, 1 << 23, (1, 32, 5, 5)) * 2.0 ** -23).astype(np.float32)
    w = np.ones((2, 32, 5, 5), np.float32)
    w[:, 1::2] = -1.0
    w[1] *= -1.0
    out, _, _ = run(x, w, (1, 1), (0, 0))
    ref = (x.astype(np.float64) * w[0]).sum()
    # 800 terms below 2: every partial sum stays below 2^11, a float addition of them rounds by at most 2^-13
    assert abs(float(out[0, 0, 0, 0]) - ref) <= 36 * 2.0 ** -13 and out[0, 1, 0, 0] == -out[0, 0, 0, 0]


def test_infinite_and_nan_inputs_reach_every_result_of_their_windows():
    rng = np.random.default_rng(9)
    w = rng.standard_normal((40, 64, 5, 5)).astype(np.float32)
    for bad in (np.inf, -np.inf, np.nan):
        x = rng.standard_normal((1, 64, 12, 12)).astype(np.float32)
        x[0, 37, 6, 6] = bad
        out, _, _ = run(x, w, (1, 1), (2, 2))
        lost = ~np.isfinite(out[0])
        assert lost[:, 4:9, 4:9].all() and lost.sum() == 40 * 25
