"""Binary-Weight-Network convolution of more than 32 channels, whose inputs xnor_bwn_split writes as digits: words that are not full,
pixels that do not fill a wave, rows so wide that a chunk holds one word (two taps per step) or takes the digits back to parts.

Bound: as in test_bwn_digits_gpu.py, six standard deviations of random roundings; the additions are those of the form that takes most,
three per 16 channels and tap."""
import numpy as np
import pytest

from oracle import xnor_oracle as xo
from tests.test_bwn_gpu import run

pytestmark = pytest.mark.gpu

# n, c, h, w, k_out, kh, kw, stride, pad
CASES = [
    (1, 33, 1, 1, 3, 1, 1, (1, 1), (0, 0)), (3, 100, 1, 1, 70, 1, 1, (1, 1), (0, 0)),          # one pixel; a tile of many images
    (5, 48, 5, 5, 33, 3, 3, (1, 1), (1, 1)), (2, 140, 13, 10, 130, 3, 3, (2, 1), (1, 0)),      # five words: workgroups of three waves
    (2, 257, 9, 9, 40, 1, 1, (1, 1), (0, 0)), (1, 512, 14, 14, 512, 3, 3, (1, 1), (1, 1)),
    (1, 64, 9, 160, 40, 5, 5, (1, 1), (2, 2)), (1, 96, 8, 170, 70, 5, 4, (1, 1), (2, 1)),      # one word per chunk
    (1, 33, 9, 150, 20, 7, 7, (1, 1), (3, 3)), (1, 72, 9, 150, 20, 7, 7, (1, 1), (3, 3)),      # parts again
    (1, 33, 110, 150, 70, 7, 7, (1, 1), (3, 3)), (1, 40, 112, 300, 20, 3, 3, (1, 1), (1, 1)),    # in tiles of 128 x 128 and 64 x 256
    (2, 64, 92, 92, 160, 7, 7, (1, 1), (3, 3)),                                                # and of 128 x 32 where 128 x 128 does not fit
]


@pytest.mark.parametrize("case", CASES)
def test_matches_oracle(case):
    n, c, h, w, k, kh, kw, stride, pad = case
    print("case", case, flush=True)
    rng = np.random.default_rng(c + h)
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    x.flat[::13] = 0.0
    wt = rng.standard_normal((k, c, kh, kw)).astype(np.float32)
    out, alpha, _ = run(x, wt, stride, pad)
    ref = xo.bwn_conv2d(x, wt, stride, pad)
    np.testing.assert_allclose(alpha, ref["alpha"], rtol=1e-5, atol=0)
    terms, adds = wt[0].size, 3 * kh * kw * ((c + 15) // 16)
    rms, top = np.sqrt(np.mean(np.square(x, dtype=np.float64))), float(np.abs(x).max())
    bound = (ref["alpha"][None, :, None, None] * np.sqrt(terms) * 6 * 2.0 ** -24 * (np.sqrt(adds / 3) * rms + top / np.sqrt(3)) +
             1e-5 * np.abs(ref["out"]))
    assert (np.abs(out.astype(np.float64) - ref["out"]) <= bound).all()


@pytest.mark.parametrize("w,kernel,pad", [(9, 3, 1), (160, 5, 2), (150, 7, 3)])
def test_infinite_and_nan_inputs_reach_every_result_of_their_windows(w, kernel, pad):
    rng = np.random.default_rng(w)
    wt = rng.standard_normal((20, 40, kernel, kernel)).astype(np.float32)
    for bad in (np.inf, np.nan):
        x = rng.standard_normal((1, 40, 9, w)).astype(np.float32)
        x[0, 35, 4, 5] = bad
        out, _, _ = run(x, wt, (1, 1), (pad, pad))
        lost = ~np.isfinite(out[0])
        assert lost[:, 4 - pad:5 + pad, 5 - pad:6 + pad].all() and lost.sum() == 20 * kernel * kernel
