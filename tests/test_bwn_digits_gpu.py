"""Binary-Weight-Network convolution with its inputs as digits (filters of 25 taps and more take that form at any size) at the
edges of its words, K-steps and chunks, and with inputs at the ends of the float range.

The float sum of c*kh*kw terms goes through 5 additions per tap and 64 channels, each off by up to half a unit in the last place
of a partial sum, which random terms keep within about the size of the whole, sqrt(terms) * rms(x); every input is off by up to
half a unit in the last place of the largest of its 32-channel word (of 2^-106, if that is larger).  Both errors are random:
|out - ref| <= alpha * sqrt(terms) * 6 * (2^-24 * sqrt(5 * taps * ceil(c / 64) / 3) * rms(x) + 2^-24 / sqrt(3) * max |x|), six standard
deviations, plus 1e-5 * |ref| for alpha's own rounding.  Single digits are checked by the exact cases below."""
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
    terms, adds = w[0].size, 5 * w.shape[2] * w.shape[3] * ((w.shape[1] + 63) // 64)
    rms, top = np.sqrt(np.mean(np.square(x, dtype=np.float64))), max(float(np.abs(x).max()), 2.0 ** -106)
    bound = (ref["alpha"][None, :, None, None] * np.sqrt(terms) * 6 * 2.0 ** -24 * (np.sqrt(adds / 3) * rms + top / np.sqrt(3)) +
             1e-5 * np.abs(ref["out"]))
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


def run_in_digits(x, w):
    """One result pixel per image, 8 images at a time: more of them under one tile stage more than the LDS holds and take the parts."""
    both = [run(x[i:i + 8], w, (1, 1), (0, 0)) for i in range(0, len(x), 8)]
    return np.concatenate([out for out, _, _ in both])[:, :, 0, 0], both[0][1]


def signs(rng, k, c):
    return np.where(rng.standard_normal((k, c, 5, 5)) >= 0, np.float32(1), np.float32(-1))      # alpha is 1 exactly


@pytest.mark.parametrize("c", [32, 33, 70, 96])
@pytest.mark.parametrize("scale", [2.0 ** -100, 1.0, 2.0 ** 126])
def test_a_single_input_comes_through_exactly(c, scale):
    # one input with a 24-bit significand below 1.875 per window: the sums of its first digits, of the even and of the odd ones are
    # floats, the fifth completes it.  Every channel of the words takes its turn.
    rng = np.random.default_rng(c)
    x, w = np.zeros((c, c, 5, 5), np.float32), signs(rng, 40, c)
    v = ((1.0 + rng.integers(0, 7 << 20, c) * 2.0 ** -23) * np.where(rng.random(c) < 0.5, 1, -1) * scale).astype(np.float32)
    at = rng.integers(0, 5, (c, 2))
    for i in range(c):
        x[i, i, at[i, 0], at[i, 1]] = v[i]
    out, alpha = run_in_digits(x, w)
    assert (alpha == 1).all()
    expect = np.stack([v[i] * w[:, i, at[i, 0], at[i, 1]] for i in range(c)])
    assert np.array_equal(out, expect)


@pytest.mark.parametrize("scale", [2.0 ** -100, 1.0, 2.0 ** 125])
def test_what_two_equal_inputs_leave_is_exact(scale):
    # two equal 24-bit inputs whose weights cancel, and the unit in their last place, in one word: that unit is the fifth digit alone
    rng = np.random.default_rng(8)
    n, c = 60, 64
    x, w = np.zeros((n, c, 5, 5), np.float32), signs(rng, 33, c)
    for i in range(n):
        (a, b, u), (ty, tx) = rng.permutation(32)[:3] + 32 * (i % 2), rng.integers(0, 5, 2)
        x[i, [a, b], ty, tx] = (1.0 + rng.integers(0, 1 << 23) * 2.0 ** -23) * scale
        x[i, b, ty, tx] *= -1 if w[0, a, ty, tx] == w[0, b, ty, tx] else 1
        x[i, u, ty, tx] = 2.0 ** -23 * scale
    ref = np.einsum("nchw,kchw->nk", x.astype(np.float64), w.astype(np.float64))
    out, _ = run_in_digits(x, w)
    assert (np.abs(ref[:, 0]) == 2.0 ** -23 * scale).all() and np.array_equal(out[:, 0], ref[:, 0].astype(np.float32))
    # filters that add the two: integers of 26 bits in that unit, rounded to 24 by each of at most six additions
    assert (np.abs(out - ref) <= 6 * 2 * 2.0 ** -23 * scale).all()


def test_the_top_binade():
    # the digits of |x| >= 1.9375 * 2^127 stay floats; such an input is held to a unit in its last place, the others exactly
    top = 31 * 2.0 ** 123
    v = np.array([top] + [float.fromhex(h) for h in ("0x1.f00002p127", "0x1.fefffep127", "0x1.effffep127", "0x1p127", "0x1.fc1234p127",
                                                     "0x1.abcdeep127")], np.float32)
    v = np.concatenate([v, -v])
    x, w = np.zeros((len(v), 40, 5, 5), np.float32), signs(np.random.default_rng(3), 20, 40) * np.float32(0.25)
    for i, f in enumerate(v):
        x[i, 3 * i % 40, i % 5, 2] = f
        x[i, (3 * i + 1) % 40, 4, i % 5] = 1.0                             # (beside it, and below what a float sum can hold)
    out, alpha = run_in_digits(x, w)
    expect = np.stack([v[i].astype(np.float64) * w[:, 3 * i % 40, i % 5, 2] for i in range(len(v))])
    ulp = np.where(np.abs(v) >= top, 2.0 ** -23, 0)[:, None]
    assert (alpha == 0.25).all() and (np.abs(out - expect) <= ulp * np.abs(expect)).all()


@pytest.mark.parametrize("outlier", [1e2, 1e4])
def test_inputs_beside_larger_ones_keep_their_part_of_the_sum(outlier):
    # one channel of every word far above the others, and log-normal inputs: the error stays below float rounding of the
    # magnitudes that a result adds up.  Half a unit in the last place of the largest of 32, for each of the others: at most
    # 32 * 2^-24 of the word's own magnitude; the additions, 2^-24 each of partial sums below the whole magnitude.
    rng = np.random.default_rng(11)
    x = rng.standard_normal((2, 96, 9, 9)) * np.exp(rng.standard_normal((2, 96, 9, 9)))
    x[:, 5::32] *= outlier
    x, w = x.astype(np.float32), signs(rng, 24, 96)
    out, _, _ = run(x, w, (1, 1), (2, 2))
    ref, size = xo.bwn_conv2d(x, w, (1, 1), (2, 2))["out"], xo.bwn_conv2d(np.abs(x), np.abs(w), (1, 1), (2, 2))["out"]
    adds = 5 * 25 * 2
    assert (np.abs(out - ref) <= 2.0 ** -24 * (32 + adds) * size).all()


def test_infinite_and_nan_inputs_reach_every_result_of_their_windows():
    rng = np.random.default_rng(9)
    w = rng.standard_normal((40, 64, 5, 5)).astype(np.float32)
    for bad in (np.inf, -np.inf, np.nan):
        x = rng.standard_normal((1, 64, 12, 12)).astype(np.float32)
        x[0, 37, 6, 6] = bad
        out, _, _ = run(x, w, (1, 1), (2, 2))
        lost = ~np.isfinite(out[0])
        assert lost[:, 4:9, 4:9].all() and lost.sum() == 40 * 25
