"""posit<8,0> products on the 6-bit floating-point matrix cores: digits, bounds, the products that go to the int8 kernel
and what they cost, edges."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2105_00053_amd as pn
from oracle import fast
from oracle import posit_oracle as po
from paper_2105_00053_amd import build

from gpu_util import mismatches, to_dev, to_np

NAR = 0x80


def test_digits_of_every_pattern():
    """h and l rebuild the value of every pattern but +-32, +-64 (flagged, zero digits) and NaR, with the bounds the exactness
    argument uses: |h| <= 48, |l| <= 16, and l = 0 from 4.0 (256 units) on."""
    L = ctypes.CDLL(build.HOSTCHECK)
    out = np.zeros(6, dtype=np.int32)
    for p in range(256):
        L.hostcheck_p8_f6(ctypes.c_uint32(p), out.ctypes.data_as(ctypes.c_void_p))
        flags, h, l, hh, ll, v = out.tolist()
        if p == NAR:
            assert (flags, h, l, hh, ll) == (1, 0, 0, 0, 0)
        elif abs(po.decode(p, po.P8)) >= 32:
            assert (flags, h, l, hh, ll) == (2, 0, 0, 0, 0)
        else:
            assert flags == 0 and v == po.decode(p, po.P8) * 64
            assert 32 * h + l == v and hh == h * h and ll == l * l
            assert abs(h) <= 48 and abs(l) <= 16 and (l == 0 or abs(v) < 256)


def _operands(kind, M, N, K):
    """Patterns of A (M x K) and B (K x N)."""
    rng = np.random.default_rng([17, M, N, K])
    if kind == "patterns":  # whole range of the format, +-32 and +-64 among it
        A, B = (rng.integers(0, 256, s, dtype=np.uint8) for s in ((M, K), (K, N)))
        A[A == NAR] = 1
        B[B == NAR] = 255
        return A, B
    if kind == "large":  # 16 and 24 everywhere: digits exist, the sums of a tile do not fit binary32
        A, B = (rng.choice(np.array([0x7C, 0x7D, 0x84, 0x83], np.uint8), s) for s in ((M, K), (K, N)))
        return A, B
    A, B = (fast.round_from_float(rng.standard_normal(s).astype(np.float32), "p8") for s in ((M, K), (K, N)))
    if kind == "one sign":  # every product positive: the largest sums the bound admits for such data
        A, B = (np.where(x >= NAR, (256 - x.astype(np.int32)), x).astype(np.uint8) for x in (A, B))
    elif kind == "some":
        A[[5, 140, 1000], [0, K - 1, 7]] = 0x81, 0x7E, 0x7F
    elif kind == "special":  # NaR at the corners, one value without digits in each operand
        A[0, 0] = A[M - 1, K - 1] = A[130, K // 2] = NAR
        B[0, 129] = B[K - 1, N - 1] = NAR
        A[300, 5] = 0x7F
        B[K - 1, 700] = 0x82
    return A, B


@pytest.mark.gpu
@pytest.mark.parametrize("kind,M,N,K,ta,tb,bias,fout", [
    ("normal", 2048, 2048, 256, False, False, False, "p8"),     # the smallest size each way: one chunk of bounds
    ("normal", 1921, 2047, 257, True, False, True, "p8"),       # one row, one index into the last tile and block; odd pitches
    ("normal", 2050, 1999, 321, False, True, True, "p16"),      # two chunks, another output format
    ("normal", 2048, 2049, 575, True, True, False, "p8_2"),
    ("one sign", 2048, 2048, 4096, False, False, False, "p8"),
    ("special", 2176, 1921, 511, False, False, True, "p8"),
    ("special", 2048, 2050, 448, True, True, False, "p16"),
    ("large", 2048, 2048, 1024, False, False, False, "p16"),
    ("patterns", 2048, 2048, 300, False, True, True, "p8"),
    ("special", 2048, 2048, 2000, False, False, True, "p16"),   # refused from the second chunk and the last on
    ("some", 2048, 2048, 700, True, False, True, "p8"),         # values without digits in the first and last chunk
    ("special", 4500, 4000, 300, False, False, False, "p8"),    # more workgroups than decide: the last ones look at what the others found
    ("normal", 4300, 2200, 300, True, False, True, "p8"),       # more than 32 tiles of rows
    ("normal", 2048, 2048, 7168, False, False, False, "p8"),    # the longest reduction, and the first beyond it
    ("normal", 2048, 2048, 7169, False, False, False, "p8"),
])
def test_products_on_the_6_bit_matrix_cores(kind, M, N, K, ta, tb, bias, fout):
    A, B = _operands(kind, M, N, K)
    b = None
    if bias:
        b = fast.round_from_float(np.random.default_rng(5).standard_normal(N).astype(np.float32), "p8")
        b[[3, N - 1]] = NAR, 0x7F
    C = pn.posit_gemm(to_dev(A.T if ta else A), to_dev(B.T if tb else B), "p8", fout, trans_a=ta, trans_b=tb, bias=None if b is None else to_dev(b))
    rows = np.unique(np.concatenate([np.arange(4), np.arange(126, 134), [300], np.arange(M - 3, M), np.random.default_rng(1).integers(0, M, 16)]))
    want, _ = fast.gemm(np.ascontiguousarray(A[rows]), B, "p8", fout, bias=b)
    assert len(mismatches(to_np(C, fout)[rows], want)) == 0


@pytest.mark.gpu
def test_one_value_without_digits_costs_no_more_than_all():
    """A product that the 6-bit kernel has to refuse is refused before it is multiplied: one +-64 among N(0, 1) operands takes no
    longer than patterns at random, which are refused everywhere."""
    rng = np.random.default_rng(3)
    one = [fast.round_from_float(rng.standard_normal((4096, 4096)).astype(np.float32), "p8") for _ in range(2)]
    one[0][1234, 321] = 0x7F
    sets = [[to_dev(x) for x in one], [to_dev(x) for x in _operands("patterns", 4096, 4096, 4096)]]
    out = torch.empty((4096, 4096), dtype=torch.uint8, device="cuda")
    times = [[], []]
    for _ in range(6):
        for (A, B), of in zip(sets, times):
            start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            for i in range(11):  # the first one untimed
                if i == 1:
                    start.record()
                pn.posit_gemm(A, B, "p8", "p8", out=out)
            stop.record()
            stop.synchronize()
            of.append(start.elapsed_time(stop))
    assert min(times[0]) < 1.1 * min(times[1])  # 1.4 when the product was taken twice, 0.96 since
