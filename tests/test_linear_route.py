"""The rules that give fully connected layers to the few-rows kernel and tiles to the words kernel (csrc/linear_route.h), compiled for the host and held
against times measured on an MI355X (back to back, us): no layer goes to a form that is clearly the slower one (no GPU)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# rows, filters, features (up to three packed words), few-rows kernel, matrix-core convolution
MEASURED_SHORT = [
    # few filters: the workgroup's 16 filter places are paid for whether they are used or not
    (8192, 4, 64, 13.2, 4.2), (16384, 1, 64, 23.8, 4.5), (32768, 1, 64, 44.1, 4.7), (2048, 8, 96, 3.2, 4.3),
    (300, 100, 96, 3.6, 4.3), (9000, 3, 96, 7.1, 4.7), (64, 512, 32, 3.3, 4.2), (1000, 30, 40, 5.1, 4.2),
]
# rows, filters, features (four words and more), few-rows kernel, linear_words_kernel
MEASURED = [
    (32768, 1, 512, 30.0, 3.7), (8192, 4, 1536, 8.9, 3.0), (65535, 1, 2048, 55.1, 7.2), (16384, 4, 3072, 15.4, 4.1),
    (65535, 2, 4096, 55.4, 11.3), (2048, 1, 512, 4.0, 2.7), (2048, 1, 9216, 4.0, 4.4), (16384, 4, 9216, 16.4, 6.7),
    (32768, 4, 8192, 29.3, 10.1), (16384, 4, 6176, 16.8, 5.6), (2048, 10, 25088, 7.3, 7.5), (8, 8192, 2368, 7.8, 3.3),
    (1024, 64, 2112, 8.0, 3.2), (128, 1024, 4160, 13.9, 3.7), (16, 8192, 8256, 23.9, 4.5), (4096, 32, 4128, 10.6, 3.8),
    (64, 1536, 12352, 18.6, 5.1), (128, 384, 3136, 6.4, 3.5), (128, 1000, 4096, 9.9, 3.8), (4096, 32, 5120, 9.6, 3.9),
    (64, 2048, 6144, 9.7, 4.0), (128, 1000, 9216, 9.9, 4.7), (1, 4096, 9216, 2.6, 4.4), (8, 4096, 9216, 4.1, 4.4),
    (1, 32768, 2048, 4.5, 4.3), (1, 65536, 4096, 7.6, 9.6), (3, 4096, 512, 3.1, 2.8), (4, 32768, 4096, 9.6, 5.5),
    (33, 1000, 2048, 4.3, 3.1), (128, 1000, 131072, 156.7, 29.7), (32, 4096, 9216, 9.4, 4.5), (64, 4096, 9216, 16.9, 4.7),
    (128, 4096, 9216, 31.1, 6.2), (256, 4096, 9216, 59.8, 8.3), (256, 100, 4096, 4.0, 3.6), (256, 100, 9216, 4.0, 4.4),
    (64, 1000, 25088, 12.8, 7.5), (16, 1000, 1024, 3.2, 2.9), (8, 4096, 4096, 4.1, 3.5), (4, 4096, 4096, 3.2, 3.5),
    (1, 1000, 100, 2.5, 2.7), (2, 4096, 9216, 2.8, 4.4), (4, 4096, 9216, 3.1, 4.4), (1, 10, 97, 2.2, 2.5),
    (758, 2, 15031, 4.9, 5.4), (16, 12, 896, 2.5, 2.6), (1230, 2, 3409, 3.2, 3.4), (24, 1, 896, 2.7, 2.5),
    (216, 60, 3288, 2.9, 3.4), (3, 4835, 240, 3.6, 2.9), (673, 2, 712, 2.8, 2.7), (27, 2, 117, 2.6, 2.5),
    (8, 75, 248, 2.6, 2.7), (12, 24, 1152, 2.6, 2.7), (334, 1, 3188, 2.8, 3.3), (1, 682, 139, 2.4, 2.7),
    (27, 11, 384, 2.5, 2.6), (7, 101, 179, 2.9, 2.7), (30, 34, 768, 2.7, 2.8), (7, 19, 1920, 2.5, 2.8),
    (85, 77, 256, 2.7, 2.8), (21, 37, 146, 2.5, 2.7), (512, 21, 128, 3.2, 2.8), (6, 24, 2289, 2.5, 2.9),
    (6, 4399, 3840, 4.1, 3.5), (2, 18, 2321, 2.4, 2.8), (88, 150, 98, 3.2, 2.9),
]
# the same against the vector-ALU convolution, for callers without the matrix image
MEASURED_NO_IMAGE = [
    (8192, 4, 64, 13.2, 6.1), (32768, 1, 512, 30.8, 7.4), (32768, 2, 2048, 30.1, 18.8), (65535, 2, 4096, 55.8, 33.4),
    (8192, 1, 32, 6.8, 5.6), (1, 4096, 4096, 2.5, 45.0),
]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, so = d / "route.cpp", str(d / "route.so")
    src.write_text('#include "linear_route.h"\n'
                   'extern "C" int route(int n, int k, int c, int image) '
                   '{ return image && c > 96 ? xnor::linear_few_rows_ahead_of_words(n, k, c, (c + 31) / 32)\n'
                   '                         : xnor::linear_popcount_route(n, k, c, (c + 31) / 32, image != 0); }\n'
                   'extern "C" int tile(int n, int k) '
                   '{ const auto t = xnor::linear_words_tile(n, k); return 10 * t.filters + t.rows; }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1603_05279_amd", "csrc"), str(src), "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("image,table", [(1, MEASURED), (1, MEASURED_SHORT), (0, MEASURED_NO_IMAGE)])
def test_no_layer_goes_to_the_clearly_slower_form(lib, image, table):
    for n, k, c, few_rows, other in table:
        took, best = (few_rows, other) if lib.route(n, k, c, image) else (other, few_rows)
        assert took <= 1.1 * best, (n, k, c, took, best)


def test_limits(lib):
    assert not lib.route(65536, 1, 9216, 1) and not lib.route(65536, 1, 96, 1)       # rows are the y extent of the grid
    assert lib.route(2, 16384, 64, 1) and not lib.route(2, 16400, 64, 1)
    assert lib.route(2, 32768, 2048, 0) and not lib.route(2, 32784, 2048, 0)
    assert lib.route(2, 65536, 4096, 0) and not lib.route(2, 65552, 4096, 0)
    for k in (1, 15_000_000, 2**31 - 1):                            # (no overflow)
        for c in (96, 97, 2**24 - 33):
            assert not lib.route(2**31 - 1, k, c, 1)
    assert not lib.route(4, 15_000_000, 97, 1) and not lib.route(65535, 65535, 2**24 - 33, 1)


# us: 1 x 1 / 2 x 1 / 2 x 2 tiles of 32 filters x rows, 9216 and 4096 features
@pytest.mark.parametrize("n,k,times", [(64, 4096, (4.9, 6.0, 7.8)), (128, 4096, (7.3, 6.5, 8.3)), (256, 4096, (11.9, 10.4, 9.1)),
                                       (256, 1000, (4.2, 4.6, 5.7))])
def test_tiles_of_the_words_kernel(lib, n, k, times):
    assert dict(zip((11, 21, 22), times))[lib.tile(n, k)] == min(times)


def test_tile_limits(lib):
    for n, k in ((1, 1), (2**30 - 1, 1), (1, 15_000_000), (2**30 - 1, 15_000_000)):          # (no overflow)
        assert lib.tile(n, k) in (11, 21, 22)
