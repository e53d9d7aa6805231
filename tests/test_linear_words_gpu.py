"""Fully connected layers on the matrix cores from packed words in registers: integers and results bit for bit against the oracle's
integers, at the edges of its word groups (eight words, the last load moved back), rows, filters and tiles (32 x 32, 64 x 32, 64 x 64)."""
import numpy as np
import pytest
import torch

from oracle import xnor_oracle as xo
from paper_1603_05279_amd import xnor
from tests.helpers import ATOL, RTOL, to_dev
from tests.test_bingrad_gpu import check as check_backward, run as run_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 97, 1), (33, 128, 31), (31, 129, 33), (64, 255, 66), (65, 256, 30), (40, 257, 7), (17, 512, 64), (96, 1000, 100),      # 4 to 9, 16, 32 words
    (300, 64 * 32 + 5, 200), (50, 67 * 32, 129), (70, 9216, 130),                             # several groups per wave
    (128, 130, 4096), (100, 300, 4090), (256, 97, 4096), (250, 353, 4093), (513, 2100, 2050),  # 64 x 32 and 64 x 64 tiles, several rounds
])
def test_matches_oracle(shape):
    b, f, o = shape
    rng = np.random.default_rng(b + f + o)
    x = rng.standard_normal((b, f)).astype(np.float32)
    w = (0.01 * rng.standard_normal((o, f))).astype(np.float32)
    r = xo.binary_linear(x, w)
    pw = xnor.PackedWeights(to_dev(w.reshape(o, f, 1, 1)))
    desc = xnor.make_desc(b, f, 1, 1, o, 1, 1)
    bufs = xnor.ConvBuffers(desc)
    xnor.xnor_binactiv(to_dev(x).reshape(b, f, 1, 1), None, None, bufs.xbits, bufs.A, None, desc)
    for algo in ("mfma_f4", "auto"):
        out = torch.full((b * o + 1,), float("nan"), device="cuda")
        dot = torch.full((b * o + 1,), 7, dtype=torch.int32, device="cuda")
        xnor.xnor_linear(bufs.xbits, pw.wbits, pw.wmfma, bufs.A, pw.alpha, out[:-1].view(b, o), dot[:-1].view(b, o), b, f, o,
                         xnor.ALGOS[algo])
        assert np.array_equal(dot[:-1].view(b, o).cpu().numpy(), r["dot"]), algo
        expect = r["dot"].astype(np.float32) * bufs.A.cpu().numpy().reshape(b, 1) * pw.alpha.cpu().numpy().reshape(1, o)
        assert np.array_equal(out[:-1].view(b, o).cpu().numpy(), expect), algo
        np.testing.assert_allclose(out[:-1].view(b, o).cpu().numpy(), r["out"], rtol=RTOL, atol=ATOL)
        assert torch.isnan(out[-1]) and dot[-1] == 7


@pytest.mark.parametrize("algo", ["mfma_f4", "auto"])
def test_backward_of_a_fully_connected_layer(algo):
    # the scale is one value per image, which here is a row
    n, c, k = 70, 300, 200
    rng = np.random.default_rng(3)
    g = rng.standard_normal((n, k, 1, 1)).astype(np.float32)
    w = (0.05 * rng.standard_normal((k, c, 1, 1))).astype(np.float32)
    alpha = rng.uniform(0.5, 1.5, k).astype(np.float32)
    check_backward(run_backward(g, w, None, alpha, (1, 1), (0, 0), algo), g, w, None, alpha, (1, 1), (0, 0))
