"""The older product kernels that the matrix-core ones have left few calls to, at sizes and pitches that still reach them (asserted where sizes decide it), against the C++ oracle."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, mismatches, rand_patterns, to_dev, to_np
from test_host_logic import CODE, hc  # noqa: F401

# 24 the 64 x 64 kernel of the vector ALU (its second size in slices), 25 the 128 x 128 one, 27 byte gather, 31 two buckets of posit<16,1>, 32 operands decoded once, 33 the general kernel
SIZES = [("p8", 2000, 1700, 200, 24), ("p8", 100, 1300, 8200, 24), ("p8", 4200, 4100, 160, 25), ("p8", 2111, 1703, 100, 25), ("p8", 253, 16, 16986, 27), ("p8_1", 253, 16, 16986, 27),
         ("p8_2", 253, 16, 16986, 27), ("p16", 129, 388, 19986, 31), ("p10_1", 493, 133, 17199, 32), ("p10_2", 171, 427, 12435, 32), ("p12_1", 434, 153, 16658, 32),
         ("p12_2", 265, 261, 12375, 32), ("p16", 1945, 270, 9, 33), ("p12_1", 1400, 1333, 16, 33), ("p12_2", 1129, 862, 16, 33)]


@pytest.mark.parametrize("fmt,M,N,K,route", SIZES)
def test_sizes_that_reach_the_older_kernels(hc, fmt, M, N, K, route):  # noqa: F811
    hc.hostcheck_gemm_route.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int]
    assert hc.hostcheck_gemm_route(CODE[fmt], M, N, K, 0) == route


def _rows(M):
    return [(0, min(4, M)), (M // 2, M // 2 + 2), (max(0, M - 3), M)]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,N,K,route", SIZES)
@pytest.mark.parametrize("order", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_products(fmt, M, N, K, route, order):
    """A row and a column of maxpos (past the range of posit<8,0>'s quire), NaR on either side, a bias."""
    ta, tb = order
    rng = np.random.default_rng(K)
    A, B = (rand_patterns(rng, s, fmt, special=0.01, allow_nar=False) for s in ((M, K), (K, N)))
    bias, nar = rand_patterns(rng, (N,), fmt, allow_nar=False), 1 << (BITS[fmt] - 1)
    A[0], A[1], B[:, 0], B[:, 1] = nar - 1, nar + 1, nar - 1, nar - 1
    B[:K // 2, 1] = nar - 2
    A[M - 1, K - 1] = B[K // 2, N - 1] = nar
    Ain, Bin = (np.ascontiguousarray(A.T) if ta else A), (np.ascontiguousarray(B.T) if tb else B)
    got = to_np(pn.posit_gemm(to_dev(Ain), to_dev(Bin), fmt, fmt, trans_a=bool(ta), trans_b=bool(tb), bias=to_dev(bias)), fmt)
    for rows in _rows(M):
        want, _ = fast.gemm(Ain, Bin, fmt, fmt, trans_a=bool(ta), trans_b=bool(tb), bias=bias, rows=rows)
        assert len(mismatches(got[rows[0]:rows[1]], want[rows[0]:rows[1]])) == 0, rows


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", ["p8", "p8_2", "p10_2", "p16", "p32"])
def test_operand_beyond_two_gigabytes(fmt):
    """A pitch that puts the last rows beyond the 32-bit offsets of the kernels straight from the patterns."""
    rng = np.random.default_rng(3)
    M, N, K, ld = 40, 64, 70, (1 << 31) // 32 + 8
    A, B = rand_patterns(rng, (M, K), fmt, allow_nar=False), rand_patterns(rng, (K, N), fmt, allow_nar=False)
    Bd = to_dev(B)
    Ad, C = torch.empty((M, ld), dtype=Bd.dtype, device="cuda"), torch.empty((M, N), dtype=Bd.dtype, device="cuda")
    Ad[:, :K] = to_dev(A)
    L, ptr = pn.load(), lambda t: ctypes.c_void_p(t.data_ptr())
    need = L.posit_gemm_workspace(CODE[fmt], CODE[fmt], 0, 0, M, N, K)
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.posit_gemm(stream, CODE[fmt], CODE[fmt], 0, 0, M, N, K, ptr(Ad), ld, ptr(Bd), N, None, ptr(C), N, ptr(ws), need) == 0
    want, _ = fast.gemm(A, B, fmt, fmt)
    assert len(mismatches(to_np(C, fmt), want)) == 0
