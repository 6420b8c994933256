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


def _wide_paddings():
    """Layers with paddings of thousands of rows or columns: strides that keep the output small, and stride 1."""
    out = []
    for pad in (1, 4000, 16383, 16385, 32767, 32769, 40000, 49151, 49152, 65535, 70001):
        st = max(1, pad // 2)
        for h, k in ((8, 128), (300, 128)):
            out.append(binding.ConvDesc(64, 16, h, 8, k, 3, 3, pad, 1, st, 1))
            out.append(binding.ConvDesc(64, 16, 8, h, k, 3, 3, 1, pad, 1, st))
            out.append(binding.ConvDesc(1, 16, h, 8, 32, 3, 3, pad, 1, 1, 1))
            out.append(binding.ConvDesc(1, 16, 8, h, 32, 3, 3, 1, pad, 1, 1))
    out.append(binding.ConvDesc(1, 8, 16384, 1, 64, 3, 1, 65534, 0, 1, 1))  # in 16 bits this padding is two rows below the taps
    out.append(binding.ConvDesc(2, 700, 1, 16000, 64, 1, 1, 8000, 0, 200, 1))
    return out


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("fmt", ["p8"] + DIGIT_FORMATS)
def test_gathers_stay_within_their_integers(hc, fmt, which):  # noqa: F811
    """What the gathering kernels rely on: a tap's offsets survive 16 bits, the rows that stand for "no pixel" stay outside, and
    every address, border included, fits 32 bits."""
    out, served = (ctypes.c_int64 * 12)(), 0
    hc.hostcheck_conv_gather_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    for d in _wide_paddings() + _bw_layers():
        if not hc.hostcheck_conv_gather_plan(CODE[fmt], which, ctypes.byref(d), out):
            continue
        served += 1
        NI, HI, WI, HO, WO, R, S, offh, offw, sh, sw, unit = out[:]
        taps = [(-offh, R - 1 - offh), (-offw, S - 1 - offw)]
        for lo, hi in taps:
            assert -32768 <= lo and hi < 0x7FFF, (d.pad_h, d.pad_w)
            assert -40000 + hi < 0
        assert HI <= 0x7FFF
        far = (((NI - 1) * HI + (HO - 1) * sh) * WI + (WO - 1) * sw) * unit
        assert far + max(0, taps[0][1] * WI + taps[1][1]) * unit < 1 << 31
        assert (taps[0][0] * WI + taps[1][0]) * unit > -(1 << 31)
    assert served > 100


def test_posit8_0_layers_of_many_channels_stay_on_the_matrix_cores(hc):  # noqa: F811
    out = (ctypes.c_int64 * 12)()
    hc.hostcheck_conv_gather_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    served = lambda c, k: hc.hostcheck_conv_gather_plan(CODE["p8"], 0, ctypes.byref(binding.ConvDesc(43, c, 14, 14, k, 1, 1, 0, 0, 1, 1)), out)  # noqa: E731
    assert served(4096, 16) and served(4097, 65) and served(8192, 256)
    assert not served(4097, 64) and not served(8193, 256)


@pytest.mark.parametrize("fmt,which,layer,served", [
    ("p8_1", 1, (64, 16, 16, 16, 16, 1), False), ("p8_2", 1, (64, 32, 16, 16, 32, 1), False), ("p8_1", 0, (32, 1, 32, 32, 32, 7), False),
    ("p8_2", 1, (32, 32, 16, 16, 1, 7), False), ("p8_1", 2, (1, 64, 64, 64, 64, 3), False), ("p8_1", 2, (130, 124, 53, 53, 24, 1), False),
    ("p8_1", 1, (128, 32, 32, 32, 32, 3), True), ("p8_2", 0, (128, 3, 32, 32, 32, 3), True), ("p8_2", 1, (64, 16, 16, 16, 16, 3), True),
    ("p8_1", 2, (128, 64, 16, 16, 64, 3), True), ("p8_2", 2, (2, 64, 64, 64, 64, 3), True), ("p16", 1, (64, 16, 16, 16, 16, 1), True)])
def test_layers_that_stay_with_the_byte_gather_kernel(hc, fmt, which, layer, served):  # noqa: F811
    """Both sides of the rule between the 8-bit formats' two kernels, at layers measured on both."""
    n, c, h, w, k, r = layer
    d = binding.ConvDesc(n, c, h, w, k, r, r, r // 2, r // 2, 1, 1)
    if layer[0] == 130:
        d.stride_h = d.stride_w = 2
    if which == 2:
        assert (_bw_need(hc, fmt, d, 1) > 0) == served
    else:
        hc.hostcheck_conv_gather_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
        assert bool(hc.hostcheck_conv_gather_plan(CODE[fmt], which, ctypes.byref(d), (ctypes.c_int64 * 12)())) == served


@pytest.mark.parametrize("fmt", ["p8_2", "p12_1", "p16"])
@pytest.mark.parametrize("which", [0, 1])
def test_passes_of_many_outputs_fit_a_launch(hc, fmt, which):  # noqa: F811
    """2^35 outputs and more in tiles of 64 x 32 or 32 x 64: fewer than 2^32 threads in a dimension, and a workgroup for every tile."""
    hc.hostcheck_dig_conv_grid.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    hc.hostcheck_dig_conv_grid.restype = ctypes.c_int64
    out = (ctypes.c_int64 * 3)()
    for n, few, many, h in ((256, 16, 2048, 256), (200, 16, 4099, 300), (1000, 1, 2049, 181), (256, 32, 64, 64)):
        d = binding.ConvDesc(n, *((few, h, h, many) if which == 0 else (many, h, h, few)), 1, 1, 0, 0, 1, 1)
        tiles = hc.hostcheck_dig_conv_grid(CODE[fmt], which, ctypes.byref(d), out)
        x, y, z = out
        assert tiles > 0 and x * 256 < 1 << 32 and y == 1 and z < 65536 and tiles <= x * z < 1 << 31
        assert (z > 1) == (h > 100)


def _direct(hc, fmt, which, layer, with_bias=0):  # noqa: F811
    """Whether a layer (N, C, H, K, R, pad, stride) goes straight from its patterns."""
    n, c, h, k, r, pad, stride = layer
    hc.hostcheck_direct_conv_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    d = binding.ConvDesc(n, c, h, h, k, r, r, pad, pad, stride, stride)
    return bool(hc.hostcheck_direct_conv_plan(CODE[fmt], which, ctypes.byref(d), with_bias, (ctypes.c_int64 * 6)()))


@pytest.mark.parametrize("fmt,which,layer,direct", [
    ("p12_2", 0, (158, 9, 40, 54, 1, 0, 1), False), ("p12_2", 0, (285, 4, 35, 52, 1, 0, 2), False), ("p8", 1, (190, 98, 37, 7, 1, 0, 2), False),
    ("p16", 1, (12, 81, 53, 4, 1, 0, 2), False), ("p12_2", 1, (14, 50, 39, 5, 1, 0, 1), False), ("p12_2", 1, (198, 104, 24, 20, 1, 0, 1), False),
    ("p12_2", 0, (8, 3, 28, 6, 5, 2, 1), True), ("p16", 0, (5, 3, 20, 20, 1, 0, 2), True), ("p10_2", 0, (64, 3, 32, 32, 3, 1, 1), True), ("p16", 1, (32, 6, 14, 16, 5, 0, 2), True)])
def test_short_reductions_of_many_outputs_stay_with_the_general_kernel(hc, fmt, which, layer, direct):  # noqa: F811
    """Both sides of the rule at layers timed on both kernels."""
    assert _direct(hc, fmt, which, layer) == direct


@pytest.mark.parametrize("fmt,which,layer,direct", [
    ("p10_1", 2, (196, 50, 34, 8, 3, 0, 1), False), ("p12_1", 2, (21, 30, 45, 44, 3, 0, 1), False), ("p8_1", 2, (189, 41, 31, 5, 5, 0, 1), False),
    ("p12_1", 2, (133, 66, 21, 146, 1, 0, 1), False), ("p10_1", 2, (124, 7, 53, 37, 3, 0, 1), False), ("p8_1", 2, (102, 33, 32, 13, 5, 0, 1), False),
    ("p8", 2, (64, 6, 14, 16, 5, 0, 1), True), ("p16", 2, (64, 1, 28, 6, 5, 2, 1), True), ("p12_1", 2, (32, 16, 12, 16, 3, 1, 1), True), ("p8_2", 2, (64, 6, 14, 16, 5, 0, 1), True)])
def test_weight_gradients_between_the_direct_kernel_and_digit_planes(hc, fmt, which, layer, direct):  # noqa: F811
    assert _direct(hc, fmt, which, layer, 1) == direct


@pytest.mark.parametrize("fmt,which,layer,direct", [
    ("p16", 0, (99, 8, 7, 53, 5, 2, 1), False), ("p8_2", 2, (9, 46, 60, 4, 5, 0, 1), False), ("p16", 1, (12, 34, 19, 10, 3, 1, 1), False),
    ("p8_1", 1, (132, 19, 32, 97, 1, 0, 1), False), ("p16", 2, (14, 18, 40, 131, 1, 0, 1), False), ("p8_1", 2, (144, 8, 60, 5, 5, 2, 1), False),
    ("p12_1", 2, (62, 83, 25, 96, 1, 0, 1), False), ("p8_1", 1, (155, 18, 50, 114, 1, 0, 1), False), ("p8_2", 0, (71, 27, 5, 144, 1, 0, 1), False),
    ("p8_2", 0, (28, 6, 9, 120, 1, 0, 1), False), ("p8_1", 0, (235, 84, 38, 23, 1, 0, 1), False), ("p16", 0, (199, 118, 40, 42, 1, 0, 2), False),
    ("p8", 0, (104, 65, 8, 118, 5, 2, 1), False), ("p8", 1, (196, 2, 8, 126, 5, 2, 1), False), ("p8", 1, (107, 98, 5, 122, 5, 0, 1), False),
    ("p16", 0, (9, 17, 26, 5, 3, 1, 1), True), ("p8_1", 2, (259, 5, 10, 106, 3, 1, 1), True), ("p10_1", 0, (63, 4, 8, 12, 5, 2, 1), True),
    ("p8_1", 1, (11, 7, 33, 10, 3, 0, 1), True), ("p12_1", 2, (235, 24, 26, 2, 1, 0, 1), True), ("p12_1", 0, (20, 29, 38, 11, 1, 0, 1), True)])
def test_layers_between_the_direct_kernel_and_the_kernels_of_16_x_32_blocks(hc, fmt, which, layer, direct):  # noqa: F811
    """Layers timed on both, a tenth and more apart."""
    assert _direct(hc, fmt, which, layer, int(which == 2)) == direct
