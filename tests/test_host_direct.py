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
    out = (ctypes.c_int64 * 7)()
    sliced = 0
    for _ in range(2000):
        M, N, K = (int(2 ** rng.uniform(0, b)) for b in (13, 13, 18))
        if not hc.hostcheck_direct_plan(CODE[fmt], M, N, K, out):
            assert K > 11904
            continue
        variant, splits, kps, ws, limbs = out[:5]
        assert variant in (1, 2, 3, 4) and kps <= 11904
        assert kps * splits >= K > kps * (splits - 1)
        if splits > 1:
            sliced += 1
            assert variant == 1 and kps % 64 == 0 and ws == 4 * splits * (M * N * limbs + M + N) <= 26 << 20
        else:
            assert ws == 0
    assert sliced > 50
    assert not hc.hostcheck_direct_plan(CODE["p32"], 64, 64, 64, out)
