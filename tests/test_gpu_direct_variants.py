"""Every cut of the kernels that multiply straight from the patterns (direct_mfma.h) against the C++ oracle, bit for bit: 16 x 16 outputs with eight and with four waves on the
reduction, 64 x 16, 32 x 32 with planes exchanged through LDS over several steps, and slices.  The sizes are chosen by the plan and the plan is asserted, here and on the CPU, so that
new estimates cannot leave a kernel untested unnoticed."""
import ctypes

import numpy as np
import pytest

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, mismatches, rand_patterns, to_dev, to_np
from test_host_logic import CODE, hc  # noqa: F401

# eight waves, four, 64 x 16, 32 x 32, slices; None: the format's estimates choose that cut for no size
PRODUCTS = {"p8": [(59, 35, 584), (212, 327, 333), (2763, 9, 55), (502, 275, 281), (67, 70, 4101)],
            "p8_1": [(50, 42, 607), (228, 289, 324), (3171, 33, 39), (287, 728, 267), (67, 70, 4101)],
            "p8_2": [(40, 53, 581), (263, 345, 521), (901, 433, 132), (87, 6582, 279), (70, 59, 1555)],
            "p10_1": [(57, 41, 582), (180, 564, 332), (5951, 34, 16), (213, 983, 264), (40, 67, 4101)],
            "p10_2": [(57, 41, 655), (147, 439, 335), (498, 532, 130), (17, 6296, 9), (40, 67, 4101)],
            "p12_1": [(57, 41, 701), (435, 419, 336), (4468, 68, 131), (569, 370, 259), (40, 67, 4101)],
            "p12_2": [(57, 41, 673), None, (359, 392, 130), (338, 401, 138), (40, 67, 4101)],
            "p16": [(57, 41, 606), (347, 81, 520), (3893, 33, 13), (83, 1596, 271), (40, 67, 4101)]}
CASES = [(f, i) for f in PRODUCTS for i in range(5) if PRODUCTS[f][i]]

# pass, layer (N, C, H, K, R, pad, stride), cut: 3 is 64 x 16, 4 is 32 x 32
LAYERS = [("p8", 0, (3, 72, 40, 90, 2, 1, 1), 4), ("p8", 1, (10, 101, 35, 35, 2, 0, 2), 3), ("p8", 1, (7, 119, 23, 30, 3, 0, 2), 4),
          ("p8_1", 0, (23, 36, 44, 1, 2, 1, 1), 3), ("p8_1", 1, (6, 105, 39, 19, 3, 1, 2), 3), ("p8_1", 1, (18, 53, 17, 17, 4, 2, 2), 4),
          ("p8_2", 0, (45, 12, 26, 2, 4, 1, 1), 3), ("p8_2", 0, (53, 9, 6, 49, 2, 1, 1), 4), ("p8_2", 1, (28, 87, 15, 10, 4, 0, 2), 3),
          ("p10_1", 0, (27, 40, 36, 1, 2, 1, 1), 3), ("p10_1", 1, (51, 39, 18, 9, 4, 2, 2), 3), ("p10_1", 1, (1, 124, 48, 31, 3, 1, 2), 4),
          ("p10_2", 0, (1, 34, 56, 99, 2, 1, 1), 3), ("p10_2", 0, (62, 1, 8, 17, 1, 0, 1), 4), ("p10_2", 1, (25, 91, 12, 12, 4, 0, 2), 3),
          ("p12_1", 0, (33, 35, 27, 1, 2, 0, 1), 3), ("p12_1", 1, (9, 121, 23, 41, 2, 0, 2), 3), ("p12_1", 1, (41, 118, 13, 84, 2, 0, 2), 4),
          ("p12_2", 0, (13, 42, 10, 102, 2, 1, 1), 3), ("p12_2", 0, (9, 36, 13, 85, 2, 1, 1), 4), ("p12_2", 1, (22, 114, 8, 15, 3, 1, 2), 4),
          ("p16", 0, (47, 10, 21, 1, 4, 1, 1), 3), ("p16", 0, (47, 20, 14, 119, 4, 0, 2), 4), ("p16", 1, (13, 80, 24, 6, 5, 0, 2), 3), ("p16", 1, (34, 115, 6, 24, 4, 0, 1), 4)]


@pytest.mark.parametrize("fmt,cut", CASES)
def test_products_that_take_each_cut(hc, fmt, cut):  # noqa: F811
    hc.hostcheck_gemm_route.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int]
    assert hc.hostcheck_gemm_route(CODE[fmt], *PRODUCTS[fmt][cut], 0) == cut + 1
    groups = 1 if fmt in ("p10_2", "p12_2") else 2
    if cut == 3 and fmt != "p10_2":
        assert -(-PRODUCTS[fmt][cut][2] // 64) > 2 * groups  # three steps and more, the last with an idle group


def _desc(layer):
    n, c, h, k, r, pad, stride = layer
    return pn.ConvDesc(n, c, h, h, k, r, r, pad, pad, stride, stride)


@pytest.mark.parametrize("fmt,which,layer,cut", LAYERS)
def test_layers_that_take_each_cut(hc, fmt, which, layer, cut):  # noqa: F811
    hc.hostcheck_direct_conv_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    out = (ctypes.c_int64 * 6)()
    assert hc.hostcheck_direct_conv_plan(CODE[fmt], which, ctypes.byref(_desc(layer)), 0, out) and out[0] == cut


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,cut", CASES)
def test_products(fmt, cut):
    M, N, K = PRODUCTS[fmt][cut]
    rng = np.random.default_rng(M + N + K)
    nar = 1 << (BITS[fmt] - 1)
    for ta, tb in ((0, 0), (1, 1), (0, 1), (1, 0)) if M * N * K < 1 << 22 else ((0, 1), (1, 0)):
        A = rand_patterns(rng, (K, M) if ta else (M, K), fmt, special=0.02, allow_nar=False)
        B = rand_patterns(rng, (N, K) if tb else (K, N), fmt, special=0.02, allow_nar=False)
        bias = rand_patterns(rng, (N,), fmt, allow_nar=False)
        (A.T if ta else A)[M - 1, K - 1] = (B.T if tb else B)[K // 2, N - 1] = bias[0] = nar
        want, _ = fast.gemm(A, B, fmt, fmt, trans_a=bool(ta), trans_b=bool(tb), bias=bias)
        got = to_np(pn.posit_gemm(to_dev(A), to_dev(B), fmt, fmt, trans_a=bool(ta), trans_b=bool(tb), bias=to_dev(bias)), fmt)
        assert len(mismatches(got, want)) == 0, (ta, tb)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,which,layer,cut", LAYERS)
def test_layers(fmt, which, layer, cut):
    n, c, h, k, r, pad, stride = layer
    rng = np.random.default_rng(sum(layer))
    d = dict(N=n, C=c, H=h, W=h, K=k, R=r, S=r, pad_h=pad, pad_w=pad, stride_h=stride, stride_w=stride)
    o, nar = (h + 2 * pad - r) // stride + 1, 1 << (BITS[fmt] - 1)
    w = rand_patterns(rng, (k, c, r, r), fmt, special=0.02, allow_nar=False)
    if which == 0:
        x, bias = rand_patterns(rng, (n, c, h, h), fmt, special=0.02, allow_nar=False), rand_patterns(rng, (k,), fmt, allow_nar=False)
        x[n - 1, c - 1, h // 2, h // 2] = w[k - 1, 0, 0, 0] = nar
        got, want = pn.posit_conv2d_fwd(to_dev(x), to_dev(w), _desc(layer), fmt, fmt, bias=to_dev(bias)), fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias)
    else:
        dy = rand_patterns(rng, (n, k, o, o), fmt, special=0.02, allow_nar=False)
        dy[0, k - 1, o - 1, 0] = w[0, c - 1, r - 1, 0] = nar
        got, want = pn.posit_conv2d_bwd_data(to_dev(dy), to_dev(w), _desc(layer), fmt, fmt), fast.conv2d_bwd_data(dy, w, d, fmt, fmt)
    assert len(mismatches(to_np(got, fmt), want)) == 0
