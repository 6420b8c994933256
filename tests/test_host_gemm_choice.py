"""Which kernel a product goes to, without a GPU: both sides of each rule at sizes that were timed on both kernels."""
import ctypes

import pytest

from test_host_logic import CODE, hc  # noqa: F401

DIRECT = (1, 2, 3, 4, 5)  # straight from the patterns


def _route(hc, fmt, M, N, K, bias=0):  # noqa: F811
    hc.hostcheck_gemm_route.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int]
    return hc.hostcheck_gemm_route(CODE[fmt], M, N, K, bias)


@pytest.mark.parametrize("fmt,M,N,K,direct", [
    ("p12_1", 2048, 2048, 16, False), ("p16", 1024, 1024, 16, False), ("p12_2", 1129, 862, 16, False), ("p10_2", 4096, 4096, 16, False),
    ("p12_1", 4096, 4096, 24, False), ("p16", 8192, 8192, 31, False), ("p12_2", 2048, 2048, 20, False), ("p12_1", 3000, 3000, 32, False),
    ("p12_1", 1129, 862, 17, True), ("p16", 1024, 1024, 31, True), ("p10_1", 4096, 4096, 24, True), ("p10_2", 2048, 2048, 17, True),
    ("p12_2", 500, 500, 16, True), ("p16", 700, 700, 8, True), ("p12_1", 4096, 4096, 48, True), ("p16", 3000, 3000, 33, True), ("p8_2", 3000, 3000, 16, True)])
def test_short_reductions_of_many_outputs(hc, fmt, M, N, K, direct):  # noqa: F811
    assert (_route(hc, fmt, M, N, K) in DIRECT) == direct


@pytest.mark.parametrize("M,N,K,direct", [
    (8192, 8192, 16, False), (8192, 8192, 255, False), (4096, 4096, 32, False), (4096, 4096, 129, False), (2048, 2048, 32, False), (3191, 2865, 64, False),
    (16384, 16384, 64, False), (2966, 6249, 82, False), (2048, 2048, 129, False), (1448, 1448, 32, True), (1536, 1536, 200, True), (1500, 1500, 255, True),
    (1024, 1024, 16, True), (100, 20000, 200, True), (20000, 64, 255, True), (65, 65, 129, True)])
def test_posit8_0_short_reductions_of_many_outputs(hc, M, N, K, direct):  # noqa: F811
    assert (_route(hc, "p8", M, N, K) in DIRECT) == direct


@pytest.mark.parametrize("fmt", ["p8", "p8_1"])
@pytest.mark.parametrize("M,N,K,direct", [(48, 48, 4, False), (250, 250, 16, False), (128, 128, 28, False), (700, 700, 8, False), (2823, 6, 32, False), (64, 84, 24, False),
                                          (48, 48, 32, True), (250, 250, 31, True), (700, 700, 12, True), (64, 120, 400, True), (3936, 12, 224, True)])
def test_short_reductions_of_few_products(hc, fmt, M, N, K, direct):  # noqa: F811
    assert (_route(hc, fmt, M, N, K) in DIRECT) == direct


@pytest.mark.parametrize("M,N,K,route", [(811, 1936, 256, 22), (6768, 256, 272, 22), (704, 2577, 293, 22), (1026, 1359, 347, 22), (512, 512, 2048, 23), (260, 816, 2048, 23),
                                         (256, 512, 8192, 23), (256, 512, 16384, 22), (256, 512, 65536, 22), (480, 544, 32768, 22), (512, 512, 65536, 23), (640, 640, 8192, 23),
                                         (1536, 1536, 1536, 22)])
def test_posit8_0_products_that_stay_with_prepared_digits(hc, M, N, K, route):  # noqa: F811
    assert _route(hc, "p8", M, N, K) == route


@pytest.mark.parametrize("fmt,M,N,K,direct", [
    ("p10_1", 4560, 416, 224, False), ("p10_1", 3655, 397, 345, False), ("p10_1", 1872, 1120, 192, False), ("p12_1", 5431, 151, 104, False),
    ("p12_1", 333, 555, 777, True), ("p16", 48, 368, 340, True), ("p10_1", 512, 512, 512, True), ("p8_1", 512, 512, 512, True), ("p12_2", 512, 512, 512, True)])
def test_products_between_the_direct_kernel_and_digit_planes(hc, fmt, M, N, K, direct):  # noqa: F811
    assert (_route(hc, fmt, M, N, K) in DIRECT) == direct


@pytest.mark.parametrize("M,N,K,route", [
    (187, 1504, 16496, 22), (480, 608, 49792, 22), (224, 1152, 15600, 22), (219, 992, 9008, 22), (896, 320, 4096, 22), (1000, 1000, 8192, 22), (512, 512, 40000, 23),
    (320, 992, 3000, 23), (224, 1216, 2048, 23), (672, 471, 22752, 23), (544, 539, 30144, 23), (768, 1024, 8192, 23), (1000, 1000, 3000, 23), (1024, 1024, 3072, 23)])
def test_posit8_0_tiles_of_32_x_32_or_slices(hc, M, N, K, route):  # noqa: F811
    assert _route(hc, "p8", M, N, K) == route
