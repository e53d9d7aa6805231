"""Fully connected layers of few rows: the vector-ALU form against the oracle, at the edges of its lane split (16 lanes x
1, 2 or 4 words, 16 filters and two rows per workgroup) and on both sides of the rule that chooses it."""
import numpy as np
import pytest
import torch

from tests.helpers import ATOL, RTOL, to_dev
from oracle import xnor_oracle as xo
from paper_1603_05279_amd import xnor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 1, 1), (1, 32, 17), (2, 33, 16), (3, 95, 15), (1, 64 * 32, 33), (5, 129 * 32, 31),     # words: 1, 2, 3, 64, 129
    (1, 256 * 32, 64), (2, 320 * 32, 9), (3, 324 * 32 - 7, 40),        # one whole turn of 4-word lanes, one word more
    # both sides of the rule: pairs, padded rows and filters, words per load, few filters
    (257, 70, 127), (258, 70, 128), (8, 2170, 8192), (9, 2170, 8192), (8, 2100, 8192), (128, 4096, 960), (128, 4096, 961),
    (1025, 40, 3), (4099, 500, 2), (37, 1000, 1030),
])
def test_few_rows_match_oracle_and_matrix_cores(shape):
    b, f, o = shape
    rng = np.random.default_rng(7 * b + f + o)
    x = rng.standard_normal((b, f)).astype(np.float32)
    w = (0.01 * rng.standard_normal((o, f))).astype(np.float32)
    r = xo.binary_linear(x, w)
    pw = xnor.PackedWeights(to_dev(w.reshape(o, f, 1, 1)))
    desc = xnor.make_desc(b, f, 1, 1, o, 1, 1)
    bufs = xnor.ConvBuffers(desc)
    xnor.xnor_binactiv(to_dev(x).reshape(b, f, 1, 1), None, None, bufs.xbits, bufs.A, None, desc)
    got = {}
    for name in ("auto", "mfma_f4"):
        out = torch.full((b, o), float("nan"), device="cuda")
        dot = torch.zeros((b, o), dtype=torch.int32, device="cuda")
        xnor.xnor_linear(bufs.xbits, pw.wbits, pw.wmfma, bufs.A, pw.alpha, out, dot, b, f, o, xnor.ALGOS[name])
        got[name] = (out.cpu().numpy(), dot.cpu().numpy())
    assert np.array_equal(got["auto"][1], r["dot"])
    assert np.array_equal(got["auto"][0], got["mfma_f4"][0])          # the same float expression on the same integers
    np.testing.assert_allclose(got["auto"][0], r["out"], rtol=RTOL, atol=ATOL)
