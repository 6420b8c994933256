"""GPU parity of the products that go to the matrix cores straight from their patterns (direct_mfma.h) against the C++ oracle, bit for
bit: edges of tiles, k blocks and slices, the four orders, pitches and odd addresses, every format, NaR and biases."""
import numpy as np
import pytest
import torch

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, NP_DTYPE, mismatches, rand_patterns, to_dev, to_np

pytestmark = pytest.mark.gpu

FORMATS = ["p8", "p8_1", "p8_2", "p10_1", "p10_2", "p12_1", "p12_2", "p16"]


def _check(rng, fin, fout, M, N, K, ta, tb, bias=True, nar=True):
    A = rand_patterns(rng, (K, M) if ta else (M, K), fin, special=0.05, allow_nar=False)
    B = rand_patterns(rng, (N, K) if tb else (K, N), fin, special=0.05, allow_nar=False)
    b = rand_patterns(rng, (N,), fin, special=0.1, allow_nar=nar) if bias else None
    if nar:
        A[rng.integers(A.shape[0]), rng.integers(A.shape[1])] = 1 << (BITS[fin] - 1)
        B[rng.integers(B.shape[0]), rng.integers(B.shape[1])] = 1 << (BITS[fin] - 1)
    want, _ = fast.gemm(A, B, fin, fout, trans_a=ta, trans_b=tb, bias=b)
    got = to_np(pn.posit_gemm(to_dev(A), to_dev(B), fin, fout, trans_a=ta, trans_b=tb, bias=to_dev(b) if bias else None), fout)
    assert len(mismatches(got, want)) == 0, (fin, fout, M, N, K, ta, tb)


# rows and columns around 16, 32 and 64, k blocks of 64 and their remainders, one and more per wave, slices (the long ones)
SIZES = [(48, 47, 1), (33, 65, 15), (17, 130, 16), (64, 33, 17), (95, 31, 63), (49, 65, 64), (100, 81, 65), (63, 97, 511), (129, 64, 513), (1, 2100, 129),
         (2050, 3, 40), (81, 82, 577), (40, 64, 4100), (70, 31, 12001)]


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("size", SIZES)
def test_sizes(fmt, size):
    rng = np.random.default_rng(sum(size))
    i = SIZES.index(size)
    _check(rng, fmt, fmt, *size, ta=bool(i & 1), tb=bool(i & 2), bias=i % 3 != 0, nar=i % 2 == 0)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("order", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_orders_and_output_formats(fmt, order):
    rng = np.random.default_rng(7)
    for fout in ("p8", "p12_2", "p16", "p32"):
        _check(rng, fmt, fout, 70, 51, 200, *map(bool, order))


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("order", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_pitches_and_odd_addresses(fmt, order):
    """Matrices inside larger ones, starting at an odd element, through the C entry point; what lies around C stays."""
    import ctypes
    rng = np.random.default_rng(9)
    L, code, n = pn.load(), pn.binding.FORMAT_CODES[fmt], BITS[fmt]
    ta, tb = order
    M, N, K, lda, ldb, ldc = 50, 45, 150, 181, 187, 53
    A = rand_patterns(rng, (K if ta else M, lda), fmt, allow_nar=False)
    B = rand_patterns(rng, (N if tb else K, ldb), fmt, allow_nar=False)
    a, b = A[:, 3:3 + (M if ta else K)], B[:, 1:1 + (K if tb else N)]
    A[:, 0] = B[:, -1] = 1 << (n - 1)  # NaR outside
    Ad, Bd = to_dev(A), to_dev(B)
    C = torch.full((M, ldc), 0x5A, dtype=Ad.dtype, device="cuda")
    e = Ad.element_size()
    ptr = lambda t, at: ctypes.c_void_p(t.data_ptr() + at * e)
    need = L.posit_gemm_workspace(code, code, ta, tb, M, N, K)
    assert need == 0
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.posit_gemm(stream, code, code, ta, tb, M, N, K, ptr(Ad, 3), lda, ptr(Bd, 1), ldb, None, ptr(C, 1), ldc, None, 0) == 0
    torch.cuda.synchronize()
    want, _ = fast.gemm(np.ascontiguousarray(a), np.ascontiguousarray(b), fmt, fmt, trans_a=bool(ta), trans_b=bool(tb))
    got = C.cpu().numpy().reshape(-1).view(NP_DTYPE[fmt])
    inside = np.lib.stride_tricks.as_strided(got[1:], (M, N), (ldc * got.itemsize, got.itemsize))
    assert len(mismatches(inside, want)) == 0
    rest = np.ones(M * ldc, bool)
    for r in range(M):
        rest[1 + r * ldc:1 + r * ldc + N] = False
    assert (got[rest] == 0x5A).all()


@pytest.mark.parametrize("fmt", FORMATS)
def test_largest_sums(fmt):
    """maxpos and its negative throughout: the sums of all planes at their largest, the quire of posit<8,0> past its range."""
    maxpos = (1 << (BITS[fmt] - 1)) - 1
    M, N, K = 64, 64, 4000
    A, B = np.full((M, K), maxpos, NP_DTYPE[fmt]), np.full((K, N), maxpos, NP_DTYPE[fmt])
    A[1::2] = (1 << BITS[fmt]) - maxpos
    A[::4, 1] = 1
    want, _ = fast.gemm(A, B, fmt, "p32")
    assert len(mismatches(to_np(pn.posit_gemm(to_dev(A), to_dev(B), fmt, "p32"), "p32"), want)) == 0


def test_operand_beyond_two_gigabytes():
    """A pitch that puts the last rows beyond the kernel's 32-bit offsets: the kernel that served before."""
    rng = np.random.default_rng(3)
    M, N, K, ld = 40, 64, 70, 1 << 26
    A, B = rand_patterns(rng, (M, K), "p8", allow_nar=False), rand_patterns(rng, (K, N), "p8", allow_nar=False)
    Ad = torch.empty((M, ld), dtype=torch.uint8, device="cuda")
    Ad[:, :K] = to_dev(A)
    L, Bd, C = pn.load(), to_dev(B), torch.empty((M, N), dtype=torch.uint8, device="cuda")
    import ctypes
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    assert L.posit_gemm(ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), 0, 0, 0, 0, M, N, K, ptr(Ad), ld, ptr(Bd), N, None, ptr(C), N, None, 0) == 0
    want, _ = fast.gemm(A, B, "p8", "p8")
    assert len(mismatches(to_np(C, "p8"), want)) == 0


@pytest.mark.parametrize("order", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("size", [(1, 1, 1), (16, 16, 64), (17, 33, 65), (50, 47, 511), (15, 100, 513), (33, 20, 2048), (300, 500, 40), (256, 251, 2049)])
@pytest.mark.parametrize("values", ["window", "range", "zero"])
def test_p32(values, size, order):
    """posit<32,2>: tiles whose operands the planes hold, tiles that span more (both kinds in one call with "range"), and zeros."""
    rng = np.random.default_rng(sum(size))
    M, N, K = size
    ta, tb = map(bool, order)
    A, B = (fast.round_from_float(rng.standard_normal(s).astype(np.float32), "p32") if values != "zero" else np.zeros(s, np.uint32)
            for s in ((K, M) if ta else (M, K), (N, K) if tb else (K, N)))
    if values == "range":
        A[(slice(None), 0) if ta else 0] = rand_patterns(rng, (K,), "p32", allow_nar=False)
        A[-1, -1], B[0, 0] = 1, 0x7FFFFFFF
        B[-1, -1] = 0x80000000
    for fout in ("p32", "p16", "p8"):
        want, _ = fast.gemm(A, B, "p32", fout, trans_a=ta, trans_b=tb)
        got = to_np(pn.posit_gemm(to_dev(A), to_dev(B), "p32", fout, trans_a=ta, trans_b=tb), fout)
        assert len(mismatches(got, want)) == 0, fout
