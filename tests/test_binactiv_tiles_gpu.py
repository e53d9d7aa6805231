"""BinActiv: tiles within an image, the last one not full or shared out among the others, and over pixels of the whole batch, where they cross
images, of fewer than 64 pixels too (the same number of workgroups on every CU); 4, 8 and 16 waves, channels that fill no group of eight."""
import numpy as np
import pytest
import torch

from oracle import xnor_oracle as xo
from paper_1603_05279_amd import xnor
from tests.helpers import ATOL, RTOL, pack_signs_channels_last, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c,h,w", [
    (1, 1, 1, 2), (3, 7, 3, 7), (130, 9, 1, 3), (5, 64, 7, 9), (2, 57, 8, 8), (7, 191, 5, 13), (7, 185, 5, 13), (1, 1000, 2, 1),
    (256, 70, 7, 7), (255, 65, 14, 14), (64, 33, 13, 13), (200, 96, 13, 13),
    (3, 20, 8, 8), (2, 65, 9, 8), (3, 12, 5, 13), (2, 90, 1, 961), (95, 40, 10, 16), (257, 9, 8, 9),     # planes around 64 pixels, batches around 256 tiles
    (40, 256, 3, 3), (200, 70, 7, 7), (120, 33, 7, 7), (64, 512, 5, 5), (2, 300, 2, 2), (1, 40, 7, 9),     # small planes: 16 pixels, an image
    (300, 127, 8, 8), (600, 130, 8, 8), (1100, 128, 8, 8), (2100, 64, 8, 8), (520, 320, 8, 8), (515, 318, 1, 64),     # both sides of the wave counts
    (2, 7680, 1, 3), (2, 7690, 1, 3), (1, 7936, 7, 10), (3, 7940, 8, 8), (3, 8064, 1, 3),     # the widest rows of 16, 8 and 4 waves
])
@pytest.mark.parametrize("bn", [False, True])
def test_matches_oracle(n, c, h, w, bn):
    print("case", n, c, h, w, bn, flush=True)
    rng = np.random.default_rng(n + c + h)
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    x.flat[::9] = 0.0
    x.flat[4::31] = -0.0
    scale, shift = (rng.uniform(0.5, 1.5, c).astype(np.float32), (0.3 * rng.standard_normal(c)).astype(np.float32)) if bn else (None, None)
    desc = xnor.make_desc(n, c, h, w, 1, 1, 1)
    words = torch.full((n * h * w * xnor.words_per_pixel(c) + 1,), 77, dtype=torch.int32, device="cuda")
    A = torch.full((n * h * w + 1,), float("nan"), device="cuda")
    sc, sh = (to_dev(scale), to_dev(shift)) if bn else (None, None)
    xnor.xnor_binactiv(to_dev(x), sc, sh, words[:-1].view(n, h, w, -1), A[:-1].view(n, h, w), None, desc)
    _, s, A_ref = xo.binactiv(x, scale, shift)
    assert np.array_equal(words[:-1].view(n, h, w, -1).cpu().numpy().view(np.uint32), pack_signs_channels_last(s))
    np.testing.assert_allclose(A[:-1].view(n, h, w).cpu().numpy(), A_ref, rtol=RTOL, atol=ATOL)
    assert words[-1] == 77 and torch.isnan(A[-1])
