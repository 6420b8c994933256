"""The digit decomposition behind the matrix-core products of the formats other than posit<8,0> (dig_planes.h), compiled
for the host: the window chosen for a range of magnitudes holds every pattern of that range exactly, and the rounding of
the combined sums is the oracle's."""
import ctypes
from fractions import Fraction

import numpy as np
import pytest

from oracle import posit_oracle as po

from test_host_logic import BITS, CODE, _p, hc  # noqa: F401

FORMATS = ["p8_1", "p8_2", "p10_1", "p12_1", "p16", "p32"]


def _lib(L):
    vp, i64, ci, u32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_uint32
    L.hostcheck_digits.argtypes = [ci, u32, u32, ci, ci, i64, vp, vp, vp]
    L.hostcheck_round_limbs.argtypes = [ci, ci, ci, i64, vp, vp]
    return L


@pytest.mark.parametrize("nar", [0, 1])
@pytest.mark.parametrize("narrow", [0, 1])
@pytest.mark.parametrize("fmt", FORMATS)
def test_window_holds_every_pattern_of_its_range(hc, fmt, narrow, nar):  # noqa: F811
    L = _lib(hc)
    top = (1 << (BITS[fmt] - 1)) - 1
    f = po.FORMATS[fmt]
    maxs = (f.n - 2) << f.es
    rng = np.random.default_rng(len(fmt) + 2 * narrow + nar)
    plane_counts = set()
    for trial in range(60):
        lo = int(rng.integers(1, top + 1)) if trial else 1
        hi = int(rng.integers(lo, top + 1)) if trial % 3 else min(top, lo + int(rng.integers(0, max(2, top // 3))))
        if trial == 0:
            hi = top
        mags = sorted({lo, hi} | {int(v) for v in rng.integers(lo, hi + 1, size=30)})
        pats = np.array([m for m in mags] + [(1 << BITS[fmt]) - m for m in mags] + [0], dtype=np.uint32)
        digits = np.zeros((len(pats), 8), dtype=np.int8)
        base = ctypes.c_int(0)
        np_ = L.hostcheck_digits(CODE[fmt], lo, hi, nar, narrow, len(pats), _p(pats), _p(digits), ctypes.byref(base))
        plane_counts.add(np_)
        if np_ == 0:  # nothing written
            assert fmt == "p32"  # every other format fits as a whole
            continue
        assert (digits[:, np_:] == 0).all()
        for p, d in zip(pats.tolist(), digits.tolist()):
            value = Fraction(0) if p == 0 else po.decode(p, f) * Fraction(2) ** maxs
            got = sum(Fraction(x) * 256 ** i for i, x in enumerate(d)) * Fraction(2) ** base.value
            assert got == value, (fmt, hex(p), d, base.value)
            if nar:
                assert -64 <= d[np_ - 1] <= 64  # -128 is the marker
    assert len(plane_counts) >= (2 if fmt == "p32" or narrow else 1)
    nar_pattern = np.array([1 << (BITS[fmt] - 1)], dtype=np.uint32)
    digits = np.zeros((1, 8), dtype=np.int8)
    np_ = L.hostcheck_digits(CODE[fmt], 1 << (BITS[fmt] - 2), 1 << (BITS[fmt] - 2), 1, narrow, 1, _p(nar_pattern), _p(digits), ctypes.byref(ctypes.c_int(0)))
    assert digits[0, np_ - 1] == -128 and (np.delete(digits[0], np_ - 1) == 0).all()


@pytest.mark.parametrize("limbs", [3, 4, 5])
def test_rounding_of_the_sums(hc, limbs):  # noqa: F811
    L = _lib(hc)
    rng = np.random.default_rng(limbs)
    formats = {0: po.P8, 1: po.P16, 2: po.P32, 4: po.P8_2, 7: po.P12_1}
    for code, f in formats.items():
        for qfrac in (0, 37, 56, 240):
            vals = [0, 1, -1, 3, -5]
            for _ in range(200):
                b = int(rng.integers(1, 32 * limbs - 1))
                v = int.from_bytes(rng.bytes(20), "little") & ((1 << b) - 1) | (1 << b - 1)
                if rng.random() < 0.5:  # ties and their neighbours: few significant bits
                    keep = int(rng.integers(1, 34))
                    v = (v >> max(0, b - keep)) << max(0, b - keep)
                    v += int(rng.integers(-1, 2))
                vals.append(-v if rng.random() < 0.5 else v)
            q = np.array([[(v >> (32 * l)) & 0xFFFFFFFF for l in range(limbs)] for v in vals], dtype=np.uint32)
            got = np.zeros(len(vals), dtype=np.uint32)
            L.hostcheck_round_limbs(limbs, qfrac, code, len(vals), _p(q), _p(got))
            for v, g in zip(vals, got.tolist()):
                assert g == po.round_to_posit(Fraction(v) / Fraction(2) ** qfrac, f), (code, qfrac, v)


@pytest.mark.parametrize("fmt,fout", [("p8_1", "p8_1"), ("p8_2", "p12_2"), ("p10_1", "p8_2"), ("p12_1", "p12_1"), ("p16", "p16"), ("p16", "p8")])
def test_rounding_through_binary64(hc, fmt, fout):  # noqa: F811
    """Both parts at every size they can have, and biases that cancel the sum, lie on its ties or far from it."""
    L = _lib(hc)
    L.hostcheck_round_f64_parts.argtypes = [ctypes.c_int] * 3 + [ctypes.c_int64] + [ctypes.c_void_p] * 4
    f, fo = po.FORMATS[fmt], po.FORMATS[fout]
    rng = np.random.default_rng(64 + f.n + fo.n)
    qmax = 2 * ((f.n - 2) << f.es)
    for qfrac in (qmax, qmax - 7, qmax // 2, qmax // 4):
        his, los, biases = [], [], []
        for i in range(1500):
            lo = int(rng.integers(0, 1 << int(rng.integers(1, 47)))) * (1 if i & 1 else -1)
            hi = (int(rng.integers(0, 1 << int(rng.integers(1, 52)))) if i % 5 else 0) * (1 if i & 2 else -1) << 24
            bias = int(rng.integers(0, 1 << f.n)) if i % 3 else 0
            if bias == 1 << (f.n - 1):
                bias = 0
            b = Fraction(0) if bias == 0 else po.decode(bias, f) * Fraction(2) ** qfrac
            if i % 4 == 1 and abs(b) < 1 << 74:  # the bias cancels all of the sum but a few units
                hi = -(int(b) >> 24) << 24
                lo = int(rng.integers(-3, 4))
            if i % 4 == 2:  # a tie of the output format, give or take a unit
                p = int(rng.integers(1, (1 << (fo.n - 1)) - 2))
                t, u = (int(po.decode(v, fo) * Fraction(2) ** qfrac) for v in (p, p + 1))
                hi, lo = ((t + u) // 2 >> 24) << 24, ((t + u) // 2 & 0xFFFFFF) + int(rng.integers(-1, 2))
            if int(float(hi)) != hi or abs(hi) >= 1 << 76:
                hi = 0
            his.append(hi)
            los.append(lo)
            biases.append(bias)
        got = np.zeros(len(his), dtype=np.uint32)
        L.hostcheck_round_f64_parts(qfrac, CODE[fmt], CODE[fout], len(his), _p(np.array(his, dtype=np.float64)), _p(np.array(los, dtype=np.float64)),
                              _p(np.array(biases, dtype=np.uint32)), _p(got))
        for h, l, bias, g in zip(his, los, biases, got.tolist()):
            b = Fraction(0) if bias == 0 else po.decode(bias, f)
            assert g == po.round_to_posit(Fraction(h + l) / Fraction(2) ** qfrac + b, fo), (qfrac, h, l, bias)


@pytest.mark.parametrize("tiles", [1, 7, 255, 2 ** 24 - 9, 2 ** 24 - 8, 2 ** 24 - 7, 2 ** 24, 2 ** 25, 2 ** 25 + 1, 2 ** 29])
def test_every_tile_has_a_workgroup_within_the_limits_of_a_launch(hc, tiles):  # noqa: F811
    """Fewer than 2^32 threads in a dimension: outputs of 2^35 and more in tiles of 64 x 32 take a second one."""
    out = (ctypes.c_int64 * 3)()
    hc.hostcheck_dig_tile_grid.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_void_p]
    hc.hostcheck_dig_tile_grid.restype = None
    hc.hostcheck_dig_tile_grid(tiles, 3, out)
    x, y, z = out
    assert x * 256 < 2 ** 32 and y == 3 and z < 65536 and x * z >= tiles and x * z < 2 ** 31
    assert z == 1 or x % 8 == 0
    assert z > 1 or x == tiles
