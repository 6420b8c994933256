"""The plans behind the convolutions on the matrix cores, as the host computes them: what a call takes is what its workspace
query answers."""
import ctypes
import random

import pytest

from paper_2105_00053_amd import binding

from test_host_logic import CODE, hc  # noqa: F401

DIGIT_FORMATS = ["p8_1", "p8_2", "p10_1", "p12_1", "p16"]


def _bw_need(L, fmt, desc, with_bias):
    L.hostcheck_conv_bw_need.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_int]
    L.hostcheck_conv_bw_need.restype = ctypes.c_size_t
    return L.hostcheck_conv_bw_need(CODE[fmt], ctypes.byref(desc), with_bias)


def _bw_layers():
    """C R S at and beside the column tiles of 64 and 128, at most 32 output channels and more, short and long reductions; then
    layers at random."""
    out = []
    for c, r, s in ((63, 1, 1), (64, 1, 1), (65, 1, 1), (128, 1, 1), (64, 3, 3), (128, 3, 3), (7, 3, 3), (32, 2, 2), (16, 2, 2)):
        for k in (20, 32, 33, 64, 128):
            for n, h in ((128, 16), (64, 32), (32, 56), (20, 28)):
                out.append(binding.ConvDesc(n, c, h, h, k, r, s, r // 2, s // 2, 1, 1))
    rng = random.Random(3)
    for _ in range(300):
        r = rng.choice([1, 2, 3, 5])
        out.append(binding.ConvDesc(rng.randint(1, 256), rng.randint(1, 160), rng.randint(6, 56), rng.randint(6, 56), rng.randint(4, 160), r, r,
                                    rng.randint(0, r // 2), rng.randint(0, r // 2), rng.choice([1, 1, 2]), 1))
    return out


@pytest.mark.parametrize("fmt", ["p8"] + DIGIT_FORMATS)
def test_weight_gradient_fits_the_queried_workspace(hc, fmt):  # noqa: F811
    L, served = binding.load(), 0
    for d in _bw_layers():
        query = L.posit_conv2d_workspace(2, CODE[fmt], CODE[fmt], ctypes.byref(d))
        for with_bias in (0, 1):
            need = _bw_need(hc, fmt, d, with_bias)
            served += need > 0
            assert need <= query, (fmt, [getattr(d, f) for f, _ in d._fields_], with_bias)
    assert served > 300
