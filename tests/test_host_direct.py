"""The kernels that multiply straight from the patterns (direct_mfma.h), compiled for the host: digits of every pattern, and what
the plan of a product promises."""
import ctypes
from fractions import Fraction

import numpy as np
import pytest

from oracle import posit_oracle as po

from test_host_logic import BITS, CODE, _p, hc  # noqa: F401

FORMATS = ["p8", "p8_1", "p8_2", "p10_1", "p10_2", "p12_1", "p12_2", "p16"]


@pytest.mark.parametrize("fmt", FORMATS)
def test_digits_of_every_pattern(hc, fmt):  # noqa: F811
    hc.hostcheck_direct_digits.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    n, f = 1 << BITS[fmt], po.FORMATS[fmt]
    maxs = (f.n - 2) << f.es
    pats, words = np.arange(n, dtype=np.uint32), np.zeros((n, 3), dtype=np.uint32)
    planes = hc.hostcheck_direct_digits(CODE[fmt], n, _p(pats), _p(words))
    digits = words.view(np.int8).reshape(n, 12).astype(object)
    assert (digits[:, planes:] == 0).all()
    got = (digits * np.array([256 ** i for i in range(12)], dtype=object)).sum(axis=1)
    for p in range(n):
        value = Fraction(0) if p in (0, n >> 1) else po.decode(p, f) * Fraction(2) ** maxs  # zero and NaR: no digits
        assert got[p] == value, (fmt, hex(p), got[p], value)
    # one workgroup's longest reduction of the largest digits stays within int32, of 8 waves in a 64-bit word
    most = 11904 * planes * 2 ** 14
    assert most < 2 ** 31 or planes == 2


@pytest.mark.parametrize("fmt", FORMATS)
def test_slices_cover_the_reduction_and_fit_the_workspace(hc, fmt):  # noqa: F811
    hc.hostcheck_direct_plan.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]
    rng = np.random.default_rng(len(fmt))
    out = (ctypes.c_int64 * 5)()
    sliced = 0
    for _ in range(2000):
        M, N, K = (int(2 ** rng.uniform(0, b)) for b in (13, 13, 18))
        if not hc.hostcheck_direct_plan(CODE[fmt], M, N, K, out):
            assert K > 11904
            continue
        variant, splits, kps, ws, limbs = out
        assert variant in (1, 2, 3, 4) and kps <= 11904
        assert kps * splits >= K > kps * (splits - 1)
        if splits > 1:
            sliced += 1
            assert variant == 1 and kps % 64 == 0 and ws == 4 * splits * (M * N * limbs + M + N) <= 26 << 20
        else:
            assert ws == 0
    assert sliced > 50
    assert not hc.hostcheck_direct_plan(CODE["p32"], 64, 64, 64, out)


TILE = {1: (16, 16, 512), 2: (16, 16, 256), 3: (64, 16, 256)}  # rows, columns and threads of a workgroup by variant


def _threads(fmt, variant, M, N):
    tr, tc, threads = TILE.get(variant, (32, 32, 256 if fmt in ("p10_2", "p12_2") else 512))
    return -(-M // tr) * -(-N // tc) * threads


@pytest.mark.parametrize("fmt", FORMATS)
def test_outputs_beyond_one_launch_are_left_to_other_kernels(hc, fmt):  # noqa: F811
    """A dimension of a launch holds fewer than 2^32 threads: 98304 x 98304 and 131072 x 131072 outputs, thin ones, and the largest that are accepted."""
    hc.hostcheck_direct_plan.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]
    out = (ctypes.c_int64 * 5)()
    for M, N, K in ((98304, 98304, 32), (131072, 131072, 64), (65536, 65536, 64), (65536, 65535, 64), (1 << 20, 1 << 16, 20), (1 << 28, 16, 8), (1 << 28, 10, 40),
                    (1 << 30, 3, 16), (1 << 20, 1 << 19, 16)):
        if hc.hostcheck_direct_plan(CODE[fmt], M, N, K, out):
            assert _threads(fmt, out[0], M, N) < 1 << 32, (M, N, K, out[0])
    assert hc.hostcheck_direct_plan(CODE[fmt], 8192, 8192, 64, out)


class _Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("N", "C", "H", "W", "K", "R", "S", "pad_h", "pad_w", "stride_h", "stride_w")]


@pytest.mark.parametrize("fmt", FORMATS)
def test_passes_beyond_one_launch_are_left_to_other_kernels(hc, fmt):  # noqa: F811
    """As above: many positions of few channels, whose tiles hold mostly padding, and weight gradients of many channels."""
    hc.hostcheck_direct_conv_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    out = (ctypes.c_int64 * 6)()
    layers = [(4000, 1, 500, 500, 1, 3, 3, 1, 1, 1, 1), (1000, 3, 512, 512, 2, 1, 1, 0, 0, 1, 1), (1000, 2, 512, 512, 3, 1, 1, 0, 0, 1, 1),
              (8000, 1, 364, 364, 1, 1, 1, 0, 0, 1, 1), (1, 1, 1, 1, 300000000, 1, 1, 0, 0, 1, 1), (2, 1, 3, 3, 50000000, 2, 2, 0, 0, 1, 1), (1, 1048575, 1, 1, 1000, 1, 1, 0, 0, 1, 1)]
    for layer in layers:
        d = _Desc(*layer)
        rows = (d.N * (d.H + 2 * d.pad_h - d.R + 1) * (d.W + 2 * d.pad_w - d.S + 1), d.N * d.H * d.W, d.K)
        for which in range(3):
            cols = (d.K, d.C, d.C * d.R * d.S + 1)[which]
            hc.hostcheck_direct_conv_plan(CODE[fmt], which, ctypes.byref(d), 1, out)  # the cut, whether or not it is the one taken
            if out[0]:
                assert _threads(fmt, out[0], rows[which], cols) < 1 << 32, (layer, which, out[0])
    d = _Desc(16, 3, 20, 20, 8, 3, 3, 1, 1, 1, 1)
    assert all(hc.hostcheck_direct_conv_plan(CODE[fmt], which, ctypes.byref(d), 1, out) or out[0] for which in range(3))


@pytest.mark.parametrize("fmt", FORMATS)
def test_sums_of_the_longest_reduction_stay_within_int32(hc, fmt):  # noqa: F811
    """A sum has at most one pair of digits per plane, each digit at most 128 in magnitude; also for two planes."""
    hc.hostcheck_direct_digits.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p]
    n = 1 << BITS[fmt]
    pats, words = np.arange(n, dtype=np.uint32), np.zeros((n, 3), dtype=np.uint32)
    planes = hc.hostcheck_direct_digits(CODE[fmt], n, _p(pats), _p(words))
    assert planes == {"p8": 2, "p8_1": 4, "p8_2": 7, "p10_1": 5, "p10_2": 9, "p12_1": 6, "p12_2": 11, "p16": 8}[fmt]
    assert 11904 * planes * 2 ** 14 < 2 ** 31
    out = (ctypes.c_int64 * 5)()
    hc.hostcheck_direct_plan.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]
    assert hc.hostcheck_direct_plan(CODE[fmt], 300, 300, 11904, out) and not hc.hostcheck_direct_plan(CODE[fmt], 300, 300, 11905, out)
