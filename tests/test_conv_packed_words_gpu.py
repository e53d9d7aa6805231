"""The 4-bit matrix-core convolution on packed weight words, at the sizes where its staging and K loop can go wrong: every
load width of the activations (1 to 4 words), odd block counts (half a K-step), channel tails, tiles that span images, rows
and strides, given K and A, dilated inputs, and channel chunks, the last of which may lack a word."""
import numpy as np
import pytest
import torch

from paper_1603_05279_amd import xnor

pytestmark = pytest.mark.gpu

# n, c, h, w, k_out, kh, kw, stride, pad
CASES = [
    (1, 1, 1, 1, 1, 1, 1, 1, 0), (2, 33, 3, 5, 40, 1, 1, 1, 0), (70, 95, 1, 1, 33, 1, 1, 1, 0),
    (3, 96, 9, 11, 100, 3, 3, 1, 1), (11, 128, 7, 7, 130, 3, 3, 1, 1), (2, 160, 13, 6, 257, 3, 3, 2, 1),
    (5, 190, 6, 14, 64, 5, 3, (1, 2), (2, 1)), (2, 224, 10, 10, 300, 3, 3, 1, 2), (1, 256, 31, 29, 129, 3, 3, 1, 1),
    (2, 384, 13, 13, 200, 3, 3, 1, 1), (1, 512, 40, 40, 32, 5, 5, 1, 2), (1, 288, 41, 41, 40, 5, 5, 2, 2), (3, 275, 9, 12, 70, 3, 3, 1, 1),
    (2, 384, 54, 54, 33, 5, 5, 1, 2), (2, 362, 53, 53, 416, 3, 3, 1, 1), (5, 320, 31, 31, 320, 3, 3, 2, 1), (1, 330, 48, 48, 140, 3, 3, 1, 1), (1, 32, 200, 3, 70, 7, 3, (3, 1), (3, 1)),
]


def block(case, algo, given_K=False, tile=0):
    n, c, h, w, k, kh, kw, stride, pad = case
    gen = torch.Generator(device="cuda").manual_seed(c * 1000 + h)
    x = torch.randn((n, c, h, w), generator=gen, device="cuda")
    wt = torch.randn((k, c, kh, kw), generator=gen, device="cuda")
    desc = xnor.make_desc(n, c, h, w, k, kh, kw, stride, pad)
    pw, bufs = xnor.PackedWeights(wt), xnor.ConvBuffers(desc, with_dot=True)
    bufs.out.fill_(float("nan"))
    bufs.dot.fill_(-(1 << 30))
    xnor.xnor_binactiv(x, None, None, bufs.xbits, bufs.A, bufs.K if given_K else None, desc)
    xnor.set_tuning(tile)
    try:
        xnor.xnor_conv2d(bufs.xbits, pw.wbits, pw.wmfma, bufs.K if given_K else None, None if given_K else bufs.A,
                         pw.alpha, bufs.out, bufs.dot, desc, xnor.ALGOS[algo])
    finally:
        xnor.set_tuning(0)
    torch.cuda.synchronize()
    return bufs


@pytest.mark.parametrize("tile", [0, 1, 2, 4, 5, 6, 11, 13, 14])
@pytest.mark.parametrize("case", CASES)
def test_same_integers_and_floats_as_the_vector_alu(case, tile):
    print("case", case, tile, flush=True)
    given_K = tile % 2 == 1
    ref, got = block(case, "popcount", given_K), block(case, "mfma_f4", given_K, tile)
    assert torch.equal(got.dot, ref.dot)
    assert torch.equal(got.out, ref.out)               # the same two float products of the same integers


@pytest.mark.parametrize("k,tile", [(64, 6), (256, 6), (257, 9), (384, 9), (100, 9), (385, 8), (512, 8), (70, 8), (600, 9)])
def test_fused_tilings_that_hold_every_filter(k, tile):
    n, c, h = 5, 96, 9
    gen = torch.Generator(device="cuda").manual_seed(k)
    xb = torch.randint(-(1 << 31), 1 << 31, (n, h, h, c // 32), generator=gen, device="cuda", dtype=torch.int64).int()
    A = torch.rand((n, h, h), generator=gen, device="cuda")
    wt = torch.randn((k, c, 3, 3), generator=gen, device="cuda")
    sc, sh = torch.rand((k,), generator=gen, device="cuda") + 0.5, torch.randn((k,), generator=gen, device="cuda")
    pw = xnor.PackedWeights(wt)
    desc = xnor.make_desc(n, c, h, h, k, 3, 3, 1, 1)
    ws = torch.empty((max(16, xnor.conv2d_binactiv_workspace_bytes(desc)),), dtype=torch.uint8, device="cuda")
    res = []
    for t in (13, tile):
        nx = torch.full((n, h, h, xnor.words_per_pixel(k)), -1, dtype=torch.int32, device="cuda")
        An, out = torch.full((n, h, h), float("nan"), device="cuda"), torch.empty((n, k, h, h), device="cuda")
        xnor.set_tuning(t)
        try:
            xnor.xnor_conv2d_binactiv(xb, pw.wbits, pw.wmfma, None, A, pw.alpha, sc, sh, nx, An, out, ws, desc,
                                      xnor.XNOR_ALGO_MFMA_F4)
        finally:
            xnor.set_tuning(0)
        res.append((nx, An, out))
    torch.cuda.synchronize()
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][2], res[1][2])
    z = torch.abs(res[1][2].double() * sc.double().view(1, -1, 1, 1) + sh.double().view(1, -1, 1, 1)).mean(1)
    # a float sum of k positive terms: at most k roundings, and one of each z
    assert torch.allclose(res[1][1].double(), z, rtol=(k + 8) * 2.0 ** -24, atol=1e-6)


@pytest.mark.parametrize("c,k,h,stride", [(64, 96, 15, (2, 2)), (40, 33, 14, (3, 2)), (32, 160, 16, (2, 1)), (70, 512, 45, (2, 2))])
def test_dilated_input(c, k, h, stride):
    # backward convolution of a strided layer: zeros between the gradient's pixels, in one chunk of words and in several;
    # against a library convolution's transpose, whose integers float64 holds exactly
    n = 3
    gen = torch.Generator(device="cuda").manual_seed(c)
    desc = xnor.make_desc(n, c, h, h, k, 3, 3, stride, 1)
    ho, wo = xnor.output_hw(desc)
    w = torch.randn((k, c, 3, 3), generator=gen, device="cuda")
    g = torch.randn((n, k, ho, wo), generator=gen, device="cuda")
    gb = torch.empty((n, ho, wo, xnor.words_per_pixel(k)), dtype=torch.int32, device="cuda")
    gmax = torch.empty((n,), device="cuda")
    xnor.xnor_bingrad_binarize(g, None, None, gb, gmax, desc)
    wt = torch.empty((c, 9, xnor.words_per_pixel(k)), dtype=torch.int32, device="cuda")
    ones, img = torch.empty((c,), device="cuda"), torch.empty((xnor.wmfma_bytes(c, k, 3, 3),), dtype=torch.uint8, device="cuda")
    xnor.xnor_bingrad_pack_weights(w, wt, ones, img, k, c, 3, 3)
    sign = lambda t: torch.where(t >= 0, 1.0, -1.0).double().cpu()
    ref = torch.nn.grad.conv2d_input((n, c, h, h), sign(w), sign(g), stride, 1)
    for algo in ("mfma_f4", "mfma_i8"):
        gin, dot = torch.empty((n, c, h, h), device="cuda"), torch.empty((n, c, h, h), dtype=torch.int32, device="cuda")
        xnor.xnor_bingrad_conv2d(gb, wt, img, gmax, ones, torch.empty((n, h, h), device="cuda"), gin, dot, desc,
                                 xnor.ALGOS[algo])
        assert torch.equal(dot.cpu().double(), ref)
        assert torch.equal(gin, dot.float() * gmax.view(-1, 1, 1, 1))


@pytest.mark.parametrize("h", [28, 30, 31])              # with the non-temporal hint: 28 x 28 only
def test_results_larger_than_the_hint_threshold(h):
    n = (64 << 20) // (256 * 4 * h * h) + 1              # just above 64 MiB of results
    ref, got = (block((n, 64, h, h, 256, 1, 1, 1, 0), algo) for algo in ("popcount", "mfma_f4"))
    assert torch.equal(got.dot, ref.dot)
    assert torch.equal(got.out, ref.out)


# n, c, h, w, k_out, kh, kw, stride, pad: rows that the tile of the layer's size cannot stage (a smaller one does)
@pytest.mark.parametrize("case", [(64, 7, 6, 700, 300, 5, 5, 2, 0), (2, 7, 16, 560, 256, 7, 7, 1, 0), (2, 7, 8, 620, 300, 7, 7, 1, 1)])
def test_layers_whose_tile_does_not_fit_take_a_smaller_one(case):
    n, c, h, w, k, kh, kw, stride, pad = case
    ref, got = block(case, "popcount"), block(case, "mfma_f4")
    assert torch.equal(got.dot, ref.dot) and torch.equal(got.out, ref.out)
    gen = torch.Generator(device="cuda").manual_seed(c * 1000 + h)
    torch.randn((n, c, h, w), generator=gen, device="cuda")                  # (block's input and weights)
    pw = xnor.PackedWeights(torch.randn((k, c, kh, kw), generator=gen, device="cuda"))
    desc = xnor.make_desc(n, c, h, w, k, kh, kw, stride, pad)
    ho, wo = xnor.output_hw(desc)
    sc, sh = torch.rand((k,), generator=gen, device="cuda") + 0.5, torch.randn((k,), generator=gen, device="cuda")
    ws = torch.empty((xnor.conv2d_binactiv_workspace_bytes(desc),), dtype=torch.uint8, device="cuda")
    nx = torch.full((n, ho, wo, xnor.words_per_pixel(k)), -1, dtype=torch.int32, device="cuda")
    An, out = torch.full((n, ho, wo), float("nan"), device="cuda"), torch.empty((n, k, ho, wo), device="cuda")
    xnor.xnor_conv2d_binactiv(ref.xbits, pw.wbits, pw.wmfma, None, ref.A, pw.alpha, sc, sh, nx, An, out, ws, desc)
    assert torch.equal(out, ref.out)
    bits, A2 = torch.empty_like(nx), torch.empty_like(An)
    xnor.xnor_binactiv(ref.out, sc, sh, bits, A2, None, xnor.make_desc(n, k, ho, wo, 1, 1, 1))
    assert torch.equal(nx, bits)
    # two float sums of k positive terms in different orders: at most k roundings each
    assert torch.allclose(An, A2, rtol=2 * k * 2.0 ** -24, atol=0)


def packed_block(c, h, k, r, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    desc = xnor.make_desc(n, c, h, h, k, r, r, 1, r // 2)
    bits = torch.randint(-(1 << 31), 1 << 31, (n, h, h, xnor.words_per_pixel(c)), generator=gen, device="cuda", dtype=torch.int64).int()
    if c % 32:
        bits[..., -1] &= (1 << (c % 32)) - 1
    A = torch.rand((n, h, h), generator=gen, device="cuda")
    pw = xnor.PackedWeights(torch.randn((k, c, r, r), generator=gen, device="cuda"))
    ref = torch.full((n, k, h, h), float("nan"), device="cuda")
    xnor.xnor_conv2d(bits, pw.wbits, pw.wmfma, None, A, pw.alpha, ref, None, desc, xnor.XNOR_ALGO_POPCOUNT)
    sc, sh = torch.rand((k,), generator=gen, device="cuda") + 0.5, torch.randn((k,), generator=gen, device="cuda")
    return desc, bits, A, pw, ref, sc, sh


# Images whose rows under a tile do not fit two workgroups of a CU with every word (wide wave tiles: and do in two chunks); 15 words: the
# last chunk lacks one
@pytest.mark.parametrize("tile,k,n,h,r", [(1, 100, 40, 30, 3), (2, 64, 260, 16, 3), (4, 200, 32, 48, 5), (5, 256, 40, 30, 3), (6, 225, 32, 48, 5),
                                          (8, 500, 32, 48, 5), (9, 384, 32, 48, 5), (11, 33, 32, 48, 5), (13, 128, 32, 48, 5),
                                          (14, 97, 32, 48, 5)])
@pytest.mark.parametrize("c", [480, 512])
def test_fused_epilogue_on_chunks_of_channel_words(c, tile, k, n, h, r):
    print("case", c, tile, k, flush=True)
    desc, bits, A, pw, ref, sc, sh = packed_block(c, h, k, r, n, c + tile)
    nx = torch.full((n, h, h, xnor.words_per_pixel(k)), -1, dtype=torch.int32, device="cuda")
    An, out = torch.full((n, h, h), float("nan"), device="cuda"), torch.full_like(ref, float("nan"))
    ws = torch.empty((max(16, xnor.conv2d_binactiv_workspace_bytes(desc)),), dtype=torch.uint8, device="cuda")
    xnor.set_tuning(tile)
    try:
        xnor.xnor_conv2d_binactiv(bits, pw.wbits, pw.wmfma, None, A, pw.alpha, sc, sh, nx, An, out, ws, desc, xnor.XNOR_ALGO_MFMA_F4)
    finally:
        xnor.set_tuning(0)
    assert torch.equal(out, ref)
    bits2, A2 = torch.empty_like(nx), torch.empty_like(An)
    xnor.xnor_binactiv(ref, sc, sh, bits2, A2, None, xnor.make_desc(n, k, h, h, 1, 1, 1))
    assert torch.equal(nx, bits2)
    # two float sums of k positive terms in different orders: at most k roundings each
    assert torch.allclose(An, A2, rtol=2 * k * 2.0 ** -24, atol=0)


# rows under three pooled ones: tiles of 96, 160 and 192 pixels; 17 words: the last chunk lacks one
@pytest.mark.parametrize("h,r", [(28, 7), (38, 5), (60, 3)])
@pytest.mark.parametrize("c", [544, 768, 1000])
def test_pooled_epilogue_on_chunks_of_channel_words(c, h, r):
    print("case", c, h, r, flush=True)
    n, k = 3, 70
    desc, bits, A, pw, ref, _, _ = packed_block(c, h, k, r, n, c + h)
    hp = (h - 3) // 2 + 1
    pooled = torch.full((n, k, hp, hp), float("nan"), device="cuda")
    xnor.xnor_conv2d_pool(bits, pw.wmfma, None, A, pw.alpha, pooled, desc, (3, 3), (2, 2))
    assert torch.equal(pooled, torch.nn.functional.max_pool2d(ref, 3, 2))
