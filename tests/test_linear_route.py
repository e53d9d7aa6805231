"""The rule that gives fully connected layers to the few-rows kernel (csrc/linear_route.h), compiled for the host and held
against times measured on an MI355X (back to back, us): no layer goes to a form that is clearly the slower one (no GPU)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# rows, filters, features, few-rows kernel, matrix cores
MEASURED = [
    # few filters: the workgroup's 16 filter places are paid for whether they are used or not
    (8192, 4, 64, 13.2, 5.0), (16384, 1, 64, 24.3, 5.7), (32768, 1, 64, 44.9, 5.6), (32768, 1, 512, 29.6, 6.0),
    (8192, 4, 1536, 9.3, 6.5), (65535, 1, 2048, 55.4, 16.4), (16384, 4, 3072, 15.7, 9.3), (65535, 2, 4096, 55.6, 28.4),
    (2048, 1, 512, 4.2, 5.0), (2048, 1, 9216, 4.2, 11.8), (16384, 4, 9216, 16.3, 36.1), (32768, 4, 8192, 30.0, 45.9),
    (16384, 4, 6176, 18.8, 344.0), (2048, 10, 25088, 7.8, 32.3),
    # rows whose words do not divide by four: narrower loads
    (4096, 4, 64, 7.9, 5.1), (8, 8192, 2368, 8.0, 6.6), (1024, 64, 2112, 8.1, 7.0), (128, 1024, 4160, 13.9, 9.5),
    (16, 8192, 8256, 24.1, 16.7), (4096, 32, 4128, 11.2, 8.9), (64, 1536, 12352, 20.0, 281.9), (128, 384, 3136, 6.7, 8.3),
    # long rows of the pair limit
    (128, 1000, 4096, 10.4, 8.5), (4096, 32, 5120, 10.3, 9.0), (64, 2048, 6144, 10.2, 13.0), (128, 1000, 9216, 10.5, 15.8),
    # one and a few rows, the sizes the kernel is for
    (1, 4096, 9216, 2.5, 9.7), (8, 4096, 9216, 3.6, 11.0), (1, 32768, 2048, 4.7, 9.3), (1, 65536, 4096, 7.9, 29.0),
    (3, 4096, 512, 3.3, 5.0), (4, 32768, 4096, 9.4, 15.2), (33, 1000, 2048, 4.7, 6.7), (128, 1000, 131072, 152.0, 277.0),
]
# the same against the vector-ALU convolution, for callers without the matrix image
MEASURED_NO_IMAGE = [
    (8192, 4, 64, 13.2, 6.1), (32768, 1, 512, 30.8, 7.4), (32768, 2, 2048, 30.1, 18.8), (65535, 2, 4096, 55.8, 33.4),
    (8192, 1, 32, 6.8, 5.6), (1, 4096, 4096, 2.5, 45.0),
]


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("route")
    src, so = d / "route.cpp", str(d / "route.so")
    src.write_text('#include "linear_route.h"\n'
                   'extern "C" int route(int n, int k, int c, int image) '
                   '{ return xnor::linear_popcount_route(n, k, c, (c + 31) / 32, image != 0); }\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1603_05279_amd", "csrc"), str(src), "-o", so], check=True)
    return ctypes.CDLL(so).route


@pytest.mark.parametrize("image,table", [(1, MEASURED), (0, MEASURED_NO_IMAGE)])
def test_no_layer_goes_to_the_clearly_slower_form(route, image, table):
    for n, k, c, few_rows, other in table:
        took, best = (few_rows, other) if route(n, k, c, image) else (other, few_rows)
        assert took <= 1.1 * best, (n, k, c, took, best)


def test_limits(route):
    assert not route(65536, 1, 9216, 1)                          # rows are the y extent of the grid
    assert route(2, 16384, 64, 1) and not route(2, 16400, 64, 1)
    assert route(2, 32768, 2048, 1) and not route(2, 32784, 2048, 1)
    assert route(2, 65536, 4096, 1) and not route(2, 65552, 4096, 1)
    assert not route(2**31 - 1, 2**31 - 1, 2**31 - 1, 1)         # (no overflow)
