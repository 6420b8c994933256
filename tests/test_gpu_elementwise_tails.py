"""Rounding, conversion and axpy where one launch takes the vectors and what is left: sizes around a vector and a workgroup, odd addresses,
every pair of formats, against the C++ oracle, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import NP_DTYPE, mismatches, rand_patterns, to_dev, to_np

pytestmark = pytest.mark.gpu

FORMATS = ["p8", "p8_1", "p8_2", "p10_1", "p10_2", "p12_1", "p12_2", "p16", "p32"]
SIZES = [1, 3, 15, 16, 17, 255, 257, 4099]


def _at(a, shift):
    """The array on the device, starting `shift` elements behind an aligned address."""
    d = to_dev(np.concatenate([a[:1].repeat(shift), a]))
    return d[shift:]


@pytest.mark.parametrize("src", FORMATS)
@pytest.mark.parametrize("shift", [0, 1])
def test_convert(src, shift):
    rng = np.random.default_rng(5)
    for dst in FORMATS:
        for n in SIZES:
            x = rand_patterns(rng, (n,), src, special=0.1)
            assert len(mismatches(to_np(pn.posit_convert(_at(x, shift), src, dst), dst), fast.convert(x, src, dst))) == 0, (dst, n)


@pytest.mark.parametrize("dst", FORMATS)
@pytest.mark.parametrize("shift", [0, 1])
def test_round(dst, shift):
    rng = np.random.default_rng(6)
    for n in SIZES:
        x = (rng.standard_normal(n) * 10.0 ** rng.integers(-12, 12, n)).astype(np.float32)
        x[rng.integers(n)] = rng.choice([np.nan, np.inf, 0.0, -0.0])
        d = torch.from_numpy(np.concatenate([x[:1].repeat(shift), x])).cuda()[shift:]
        assert len(mismatches(to_np(pn.posit_round(d, dst), dst), fast.round_from_float(x, dst))) == 0, n


# where the kernels with formats as constants and the table take over, vectors whole and with a remainder
LARGE = [163839, 163840, 163857, 393215, 393216, 393219, 720895, 720896, 720903]


@pytest.mark.parametrize("pair", [("p12_2", "p8_2"), ("p10_2", "p8_2"), ("p12_1", "p8_1"), ("p10_1", "p8_1"), ("p8_1", "p12_1"), ("p8_2", "p8_1"), ("p8", "p10_2"), ("p8_2", "p32")])
@pytest.mark.parametrize("shift", [0, 1])
def test_convert_large(pair, shift):
    src, dst = pair
    rng = np.random.default_rng(7)
    for n in LARGE:
        x = rand_patterns(rng, (n,), src, special=0.1)
        assert len(mismatches(to_np(pn.posit_convert(_at(x, shift), src, dst), dst), fast.convert(x, src, dst))) == 0, n


@pytest.mark.parametrize("dst", ["p8_1", "p8_2", "p10_1", "p10_2", "p12_1", "p12_2"])
@pytest.mark.parametrize("shift", [0, 1])
def test_round_large(dst, shift):
    rng = np.random.default_rng(6)
    for n in LARGE[3:6]:
        x = (rng.standard_normal(n) * 10.0 ** rng.integers(-12, 12, n)).astype(np.float32)
        x[rng.integers(n, size=4)] = [np.nan, np.inf, 0.0, -0.0]
        d = torch.from_numpy(np.concatenate([x[:1].repeat(shift), x])).cuda()[shift:]
        assert len(mismatches(to_np(pn.posit_round(d, dst), dst), fast.round_from_float(x, dst))) == 0, n


@pytest.mark.parametrize("pair", [("p8", "p16", "p8"), ("p16", "p16", None), ("p16", "p32", "p16"), ("p8", "p8", None), ("p32", "p32", "p8")])
@pytest.mark.parametrize("shift", [0, 1])
def test_axpy(pair, shift):
    fx, fy, fc = pair
    rng = np.random.default_rng(8)
    for n in SIZES:
        x, y = rand_patterns(rng, (n,), fx, special=0.1), rand_patterns(rng, (n,), fy, special=0.1)
        yd = _at(y, shift)
        alpha = int(rand_patterns(rng, 1, fy, 0, allow_nar=False)[0])
        got, want = pn.posit_axpy(alpha, _at(x, shift), yd, fx, fy, fc), fast.axpy(alpha, x, y, fx, fy, fc)
        for g, w, f in zip(got if fc else (got,), want if fc else (want,), (fy, fc)):
            assert len(mismatches(to_np(g, f), w)) == 0, n
