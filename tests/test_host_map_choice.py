"""Which kernel a rounding or conversion beyond Table 1 goes to, at sizes timed on both sides of each rule."""
import ctypes

import pytest

from test_host_logic import CODE, hc  # noqa: F401

RUNTIME, TYPED, TABLE = 0, 1, 2


@pytest.mark.parametrize("src,dst,n,kernel", [
    ("f32", "p8_2", 100, RUNTIME), ("f32", "p8_2", 64 * 784, RUNTIME), ("f32", "p12_1", 262144, RUNTIME), ("f32", "p10_2", 400000, TYPED), ("f32", "p8_1", 2 ** 24, TYPED),
    ("p12_2", "p8_2", 100, RUNTIME), ("p10_1", "p8_1", 500000, RUNTIME), ("p12_1", "p8_1", 1000003, TYPED), ("p10_2", "p8_2", 2 ** 24, TYPED),
    ("p8_2", "p12_2", 100, RUNTIME), ("p8", "p8_1", 131072, RUNTIME), ("p8_1", "p12_1", 200003, TABLE), ("p8_2", "p32", 2 ** 24, TABLE), ("p12_2", "p12_1", 2 ** 24, RUNTIME)])
def test_map_choice(hc, src, dst, n, kernel):  # noqa: F811
    code = dict(CODE, f32=100)
    hc.hostcheck_map_choice.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    assert hc.hostcheck_map_choice(code[src], code[dst], n) == kernel
