"""Fused epilogue in the tiles whose 8 to 16 waves hold 32 filters each (256 x 96, 384 x 96, 256 x 32, 512 x 32 pixels): the result, the sign words and
A of the next block at the edges of their filters and pixels, against the vector-ALU convolution and the stand-alone BinActiv."""
import pytest
import torch

from paper_1603_05279_amd import xnor
from tests.test_conv_packed_words_gpu import packed_block

pytestmark = pytest.mark.gpu


# n, c, h, k, filter size; tile 0: the library's choice (each of the tiles among them)
@pytest.mark.parametrize("tile,n,c,h,k,r", [
    (3, 1, 32, 4, 1, 3), (3, 9, 70, 7, 129, 3), (3, 2, 200, 13, 255, 5), (3, 3, 96, 20, 256, 1), (9, 1, 64, 5, 33, 3), (9, 9, 100, 7, 257, 3),
    (9, 2, 33, 19, 353, 5), (9, 5, 256, 13, 384, 1), (0, 100, 64, 13, 200, 3), (0, 90, 40, 13, 320, 3),
    (7, 1, 32, 3, 1, 3), (7, 5, 70, 7, 129, 3), (7, 2, 480, 9, 255, 5), (7, 3, 96, 11, 256, 1), (10, 1, 64, 5, 33, 3), (10, 5, 100, 7, 257, 3),
    (10, 2, 33, 9, 511, 5), (10, 4, 480, 14, 512, 1), (0, 3, 64, 9, 130, 3), (0, 3, 200, 9, 400, 1),
])
@pytest.mark.parametrize("with_out", [True, False])
def test_fused_tiles(tile, n, c, h, k, r, with_out):
    print("case", tile, n, c, h, k, r, flush=True)
    desc, bits, A, pw, ref, sc, sh = packed_block(c, h, k, r, n, c + k)
    nx = torch.full((n, h, h, xnor.words_per_pixel(k)), -1, dtype=torch.int32, device="cuda")
    An, out = torch.full((n, h, h), float("nan"), device="cuda"), torch.full_like(ref, float("nan")) if with_out else None
    ws = torch.empty((max(16, xnor.conv2d_binactiv_workspace_bytes(desc)),), dtype=torch.uint8, device="cuda")
    xnor.set_tuning(tile)
    try:
        xnor.xnor_conv2d_binactiv(bits, pw.wbits, pw.wmfma, None, A, pw.alpha, sc, sh, nx, An, out, ws, desc, xnor.XNOR_ALGO_MFMA_F4)
    finally:
        xnor.set_tuning(0)
    if with_out:
        assert torch.equal(out, ref)
    bits2, A2 = torch.empty_like(nx), torch.empty_like(An)
    xnor.xnor_binactiv(ref, sc, sh, bits2, A2, None, xnor.make_desc(n, k, h, h, 1, 1, 1))
    assert torch.equal(nx, bits2)
    # two float sums of k positive terms in different orders: at most k roundings each
    assert torch.allclose(An, A2, rtol=2 * k * 2.0 ** -24, atol=0)
