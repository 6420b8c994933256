"""The older convolution kernels (dot products of posit<8,0>, byte gather, the general kernel) at layers that the matrix-core kernels leave to them, which is asserted, against the C++
oracle, bit for bit."""
import ctypes

import numpy as np
import pytest

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, mismatches, rand_patterns, to_dev, to_np
from test_host_logic import CODE, hc  # noqa: F401

FORMATS = ["p8", "p8_1", "p8_2", "p10_1", "p10_2", "p12_1", "p12_2", "p16"]
TALL = (2, 3, 33000, 1, 5, 3, 1, 1, 0, 1, 1)  # N, C, H, W, K, R, S, pad_h, pad_w, stride_h, stride_w: more rows than those kernels' coordinates hold
STRIDED = (2, 2, 65999, 1, 3, 2, 1, 0, 0, 2, 1)
CASES = [(f, w, g) for f in FORMATS for w in range(3) for g in (TALL, STRIDED)]


def _square(n, c, h, k, r, pad, stride):
    return (n, c, h, h, k, r, r, pad, pad, stride, stride)


CASES += [("p8", 0, _square(111, 1, 29, 1, 2, 0, 1)), ("p8", 0, _square(120, 1, 31, 1, 2, 1, 2)), ("p8", 1, _square(35, 1, 42, 1, 2, 1, 1)), ("p8", 1, _square(18, 14, 47, 1, 1, 0, 2)),
          ("p8_1", 0, _square(10, 1, 38, 19, 2, 1, 1)), ("p8_1", 0, _square(76, 1, 32, 24, 2, 0, 2)), ("p8_1", 1, _square(2, 1, 6, 102, 6, 1, 1)), ("p8_1", 1, _square(69, 4, 45, 1, 2, 0, 2)),
          ("p8_2", 0, _square(7, 1, 28, 1, 2, 1, 1)), ("p8_2", 1, _square(92, 65, 10, 1, 2, 0, 2)), ("p8_2", 2, _square(3, 46, 1, 109, 5, 2, 1)), ("p8_2", 2, _square(1, 103, 6, 46, 6, 0, 2)),
          ("p10_1", 0, _square(6, 1, 57, 89, 1, 0, 1)), ("p10_1", 1, _square(16, 21, 46, 1, 2, 1, 2)), ("p10_2", 0, _square(31, 1, 16, 65, 2, 1, 1)), ("p12_1", 1, _square(109, 124, 7, 1, 2, 0, 1)),
          ("p12_2", 0, _square(12, 1, 53, 33, 2, 1, 2)), ("p12_2", 1, _square(94, 49, 8, 1, 2, 0, 1)), ("p16", 0, _square(104, 1, 56, 14, 1, 0, 2)), ("p16", 1, _square(16, 28, 35, 1, 2, 1, 2))]


@pytest.mark.parametrize("fmt,which,layer", CASES)
def test_layers_that_are_left_to_the_older_kernels(hc, fmt, which, layer):  # noqa: F811
    d = pn.ConvDesc(*layer)
    hc.hostcheck_direct_conv_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    hc.hostcheck_conv_gather_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    hc.hostcheck_conv_bw_need.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_int]
    hc.hostcheck_conv_bw_need.restype = ctypes.c_size_t
    assert not hc.hostcheck_direct_conv_plan(CODE[fmt], which, ctypes.byref(d), int(which == 2), (ctypes.c_int64 * 6)())
    if which == 2:
        assert not hc.hostcheck_conv_bw_need(CODE[fmt], ctypes.byref(d), 1)
    else:
        assert not hc.hostcheck_conv_gather_plan(CODE[fmt], which, ctypes.byref(d), (ctypes.c_int64 * 12)())


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,which,layer", CASES)
def test_passes(fmt, which, layer):
    rng = np.random.default_rng(sum(layer))
    d = dict(zip(("N", "C", "H", "W", "K", "R", "S", "pad_h", "pad_w", "stride_h", "stride_w"), layer))
    desc, nar = pn.ConvDesc(*layer), 1 << (BITS[fmt] - 1)
    oh, ow = fast.out_hw(d)
    tensor = lambda *shape: rand_patterns(rng, shape, fmt, special=0.02, allow_nar=False)  # noqa: E731
    x, w, dy, bias = tensor(d["N"], d["C"], d["H"], d["W"]), tensor(d["K"], d["C"], d["R"], d["S"]), tensor(d["N"], d["K"], oh, ow), tensor(d["K"])
    x[-1, -1, d["H"] // 2, 0] = w[-1, 0, 0, 0] = dy[0, 0, -1, -1] = bias[0] = nar
    same = lambda got, want: len(mismatches(to_np(got, fmt), want)) == 0  # noqa: E731
    if which == 0:
        assert same(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, fmt, bias=to_dev(bias)), fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias))
    elif which == 1:
        assert same(pn.posit_conv2d_bwd_data(to_dev(dy), to_dev(w), desc, fmt, fmt), fast.conv2d_bwd_data(dy, w, d, fmt, fmt))
    else:
        dw, db = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), desc, fmt, fmt, with_bias=True)
        want_dw, want_db = fast.conv2d_bwd_weight(dy, x, d, fmt, fmt, with_bias=True)
        assert same(dw, want_dw) and same(db, want_db)
