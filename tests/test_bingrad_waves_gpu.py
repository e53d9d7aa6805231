"""Gradient binarisation with four and eight waves, filters that fill no group of eight, runs of several tiles, the last one not
full, and the widest word rows that LDS holds."""
import numpy as np
import pytest
import torch

from paper_1603_05279_amd import xnor
from tests.helpers import to_dev
from tests.test_bingrad_gpu import pack_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,h,w", [(3, 56, 7, 9), (2, 57, 8, 8), (5, 65, 7, 7), (2, 511, 5, 13), (1, 8160, 2, 3), (4, 7, 1, 65), (300, 40, 16, 17), (130, 72, 26, 27),
                                     (64, 72, 30, 30), (200, 17, 31, 31), (30, 100, 40, 41), (70, 64, 57, 56)])
@pytest.mark.parametrize("with_k,with_alpha", [(True, True), (False, False)])
def test_signs_and_maxima(n, k, h, w, with_k, with_alpha):
    print("case", n, k, h, w, flush=True)
    rng = np.random.default_rng(n + k)
    g = rng.standard_normal((n, k, h, w)).astype(np.float32)
    g.flat[::7] = 0.0
    g.flat[3::50] = np.nan
    K = rng.uniform(0.1, 1, (n, h, w)).astype(np.float32)
    alpha = rng.uniform(0.1, 1, k).astype(np.float32)
    gd = g * (alpha.reshape(1, k, 1, 1) if with_alpha else np.float32(1)) * (K[:, None] if with_k else np.float32(1))
    desc = xnor.make_desc(n, 3, h, w, k, 1, 1)
    bits = torch.full((n, h, w, xnor.words_per_pixel(k)), 77, dtype=torch.int32, device="cuda")
    gmax = torch.full((n,), 123.0, device="cuda")
    xnor.xnor_bingrad_binarize(to_dev(g), to_dev(K) if with_k else None, to_dev(alpha) if with_alpha else None, bits, gmax, desc)
    assert np.array_equal(bits.cpu().numpy().view(np.uint32), pack_bits(np.where(gd >= 0, 1, -1)))
    assert np.array_equal(gmax.cpu().numpy(), np.nanmax(np.abs(gd).reshape(n, -1), axis=1))
