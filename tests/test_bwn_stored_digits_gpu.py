"""Binary-Weight-Network convolution of more than 48 channels on rows of at most 64 pixels, whose inputs xnor_bwn_split writes as digits: words
that are not full, pixels that do not fill a wave, filters so tall that a chunk holds one word (two taps per step) or takes the digits back to
parts; and of wider rows, which it writes as parts.

Bound: as in test_bwn_digits_gpu.py, six standard deviations of random roundings; the additions are those of the form that takes most,
three per 16 channels and tap."""
import numpy as np
import pytest

from oracle import xnor_oracle as xo
from tests.test_bwn_gpu import run

pytestmark = pytest.mark.gpu

# n, c, h, w, k_out, kh, kw, stride, pad
CASES = [
    (1, 49, 1, 1, 3, 1, 1, (1, 1), (0, 0)), (3, 100, 1, 1, 70, 1, 1, (1, 1), (0, 0)),          # one pixel; a tile of many images
    (5, 52, 5, 5, 33, 3, 3, (1, 1), (1, 1)), (2, 140, 13, 10, 130, 3, 3, (2, 1), (1, 0)),      # five words: workgroups of three waves
    (2, 257, 9, 9, 40, 1, 1, (1, 1), (0, 0)), (1, 512, 14, 14, 512, 3, 3, (1, 1), (1, 1)),
    (1, 64, 30, 64, 40, 13, 13, (1, 1), (6, 6)), (1, 96, 31, 62, 70, 12, 11, (1, 1), (5, 5)),  # one word per chunk, of an odd and an even number of taps
    (1, 64, 30, 64, 20, 15, 15, (1, 1), (7, 7)),                                               # parts again, 128 x 32
    (9, 64, 31, 60, 70, 9, 3, (1, 1), (4, 1)), (9, 64, 64, 62, 20, 8, 7, (1, 1), (4, 3)),        # in tiles of 128 x 128 and 64 x 256
    (20, 64, 31, 60, 70, 11, 3, (1, 1), (5, 1)),                                               # and of 128 x 32 where 128 x 128 does not fit
    (1, 33, 9, 150, 20, 7, 7, (1, 1), (3, 3)), (1, 72, 9, 150, 20, 7, 7, (1, 1), (3, 3)),      # wide rows: parts
    (1, 33, 110, 150, 70, 7, 7, (1, 1), (3, 3)), (1, 40, 112, 300, 20, 3, 3, (1, 1), (1, 1)),
    (2, 64, 92, 92, 160, 7, 7, (1, 1), (3, 3)),
    (1, 64, 9, 65, 40, 5, 5, (1, 1), (2, 2)), (1, 96, 8, 66, 70, 5, 4, (1, 1), (2, 1)),        # digits made of several words of parts
    (1, 290, 12, 66, 40, 5, 7, (1, 1), (2, 3)), (1, 160, 14, 80, 100, 5, 5, (2, 2), (1, 2)),
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


@pytest.mark.parametrize("w,kernel", [(41, 3), (64, 13), (64, 15), (66, 5), (150, 7)])
def test_infinite_and_nan_inputs_reach_every_result_of_their_windows(w, kernel):
    rng = np.random.default_rng(w)
    wt, pad = rng.standard_normal((20, 70, kernel, kernel)).astype(np.float32), kernel // 2
    for bad in (np.inf, np.nan):
        x = rng.standard_normal((1, 70, 30, w)).astype(np.float32)
        x[0, 35, 14, 25] = bad
        out, _, _ = run(x, wt, (1, 1), (pad, pad))
        lost = ~np.isfinite(out[0])
        assert lost[:, 14 - pad:15 + pad, 25 - pad:26 + pad].all() and lost.sum() == 20 * kernel * kernel


@pytest.mark.parametrize("kernel", [1, 3])
@pytest.mark.parametrize("outlier", [1e2, 1e4, 1e6])
def test_what_large_inputs_that_cancel_leave(kernel, outlier):
    # Two equal large inputs in every word, which about half of the filters subtract: an input is off by at most half a unit in the last
    # place of its word's largest, 2^-24 of that one, 31 of them to a word and tap; an addition by 2^-24 of a partial sum.
    rng = np.random.default_rng(5)
    x = rng.standard_normal((2, 96, 9, 9))
    x[:, 3::32] = x[:, 17::32] = outlier * (1 + rng.random((2, 3, 9, 9)))
    x = x.astype(np.float32)
    w = np.where(rng.standard_normal((24, 96, kernel, kernel)) >= 0, np.float32(1), np.float32(-1))       # alpha is 1 exactly
    pad, adds = (kernel // 2, kernel // 2), 5 * kernel * kernel * 2
    out, _, _ = run(x, w, (1, 1), pad)
    ref, size = xo.bwn_conv2d(x, w, (1, 1), pad)["out"], xo.bwn_conv2d(np.abs(x), np.abs(w), (1, 1), pad)["out"]
    assert (np.abs(out - ref) <= 2.0 ** -24 * (31 + adds) * size).all()
