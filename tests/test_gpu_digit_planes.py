"""posit_gemm on the integer matrix cores as base-256 digit planes (every format other than posit<8,0>, (10,2), (12,2)), at
the sizes and operands where the path can go wrong: edges of tiles and k blocks, the ends of the range of shapes that
takes it, reductions cut into slices, windows at their limits, rare small values below the planes of the main loop, NaR,
all-zero operands.  Bit-exact against the oracle."""
import numpy as np
import pytest

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, NP_DTYPE, mismatches, rand_patterns, to_dev, to_np

pytestmark = pytest.mark.gpu


def _operand(rng, shape, fmt, kind):
    if kind == "uniform":  # all patterns: the widest kernel, or (posit<32,2>) the one with the quire in LDS
        return rand_patterns(rng, shape, fmt, special=0.01, allow_nar=False)
    if kind == "zero":
        return np.zeros(shape, dtype=NP_DTYPE[fmt])
    x = rng.standard_normal(shape)
    if kind == "relu":
        x = np.maximum(x, 0.0)
    elif kind == "tiny":  # a few values far below the others: k blocks that are looked at twice
        x = np.where(rng.random(shape) < 2e-4, x * 2.0 ** -13, x)
    elif kind == "scaled":
        x = x * 2.0 ** -9
    return fast.round_from_float(x.astype(np.float32), fmt)


def _check(fmt, fout, M, N, K, ta, tb, kinds, bias=False, nar=False):
    rng = np.random.default_rng(M + 3 * N + 7 * K + BITS[fmt])
    A, B = _operand(rng, (M, K), fmt, kinds[0]), _operand(rng, (K, N), fmt, kinds[1])
    nar_in, nar_out = 1 << (BITS[fmt] - 1), 1 << (BITS[fout] - 1)
    if nar:
        A[M - 1, K - 1] = A[33, 0] = nar_in
        B[K - 1, N - 1] = nar_in
    bv = None
    if bias:
        bv = _operand(rng, (N,), fmt, "uniform")
        bv[1] = nar_in
    Ain, Bin = (np.ascontiguousarray(A.T) if ta else A), (np.ascontiguousarray(B.T) if tb else B)
    got = to_np(pn.posit_gemm(to_dev(Ain), to_dev(Bin), fmt, fout, trans_a=ta, trans_b=tb, bias=None if bv is None else to_dev(bv)), fout)
    rows = np.arange(M) if M * N * K <= 1 << 26 else np.array(sorted({0, 31, 32, 33, 63, 64, M - 2, M - 1} | {int(r) for r in rng.integers(0, M, 6)}))
    want, _ = fast.gemm(np.ascontiguousarray(A[rows]), B, fmt, fout, bias=bv)
    bad = mismatches(got[rows], want)
    assert len(bad) == 0, "%s %dx%dx%d %s: %d outputs differ, first at %s" % (fmt, M, N, K, kinds, len(bad), bad[0])
    if nar:
        assert (got[M - 1] == nar_out).all() and (got[33] == nar_out).all() and (got[:, N - 1] == nar_out).all()
    return got


@pytest.mark.parametrize("fmt,M,N,K,ta,tb", [
    ("p16", 96, 96, 64, 0, 0), ("p16", 97, 129, 65, 0, 1), ("p16", 128, 191, 96, 1, 0), ("p12_1", 333, 200, 129, 1, 1),
    ("p10_1", 100, 640, 1023, 0, 0), ("p16", 100, 97, 16352, 0, 0), ("p16", 100, 97, 16353, 0, 0), ("p12_1", 300, 260, 4100, 1, 0),
    ("p8_2", 600, 390, 257, 0, 1), ("p8_1", 520, 270, 333, 1, 1), ("p8_2", 384, 400, 2048, 0, 0), ("p32", 450, 470, 256, 0, 1),
    ("p32", 449, 450, 1000, 1, 0), ("p32", 447, 452, 16352, 0, 0)])
@pytest.mark.parametrize("kinds", [("gauss", "gauss"), ("tiny", "relu"), ("uniform", "scaled")])
def test_sizes_at_the_edges(fmt, M, N, K, ta, tb, kinds):
    if K > 4096 and kinds[0] == "uniform":
        K = K // 4 + 1
    _check(fmt, fmt, M, N, K, ta, tb, kinds)


@pytest.mark.parametrize("fmt,fout,M,N,K", [("p16", "p8", 130, 140, 300), ("p16", "p32", 130, 140, 300), ("p12_1", "p12_1", 257, 100, 500),
                                            ("p10_1", "p8_2", 120, 333, 777), ("p8_2", "p12_2", 500, 520, 300), ("p8_1", "p12_1", 500, 520, 300),
                                            ("p32", "p16", 460, 455, 300)])
@pytest.mark.parametrize("kinds", [("gauss", "tiny"), ("uniform", "uniform"), ("zero", "gauss"), ("relu", "zero")])
@pytest.mark.parametrize("bias", [False, True])
def test_bias_nar_and_output_formats(fmt, fout, M, N, K, kinds, bias):
    got = _check(fmt, fout, M, N, K, 0, 0, kinds, bias=bias, nar=True)
    if "zero" in kinds and not bias:
        inner = np.delete(got, [33, M - 1], axis=0)[:, :N - 1]
        assert (inner == 0).all()


@pytest.mark.parametrize("fmt,fout,M,N,K", [("p16", "p16", 1030, 1100, 96), ("p12_1", "p16", 1030, 1100, 70), ("p10_1", "p10_1", 1030, 1100, 64),
                                            ("p8_2", "p12_2", 1030, 1100, 258), ("p8_1", "p8_1", 1030, 1100, 258), ("p8_1", "p8_1", 2050, 2100, 512)])
@pytest.mark.parametrize("up", [-10, -5, 0, 5, 12])
def test_bias_at_every_weight_of_the_sums(fmt, fout, M, N, K, up):
    """Uncut products whose sums' unit lies below minpos^2, between it and the unit of the biases, and above that; biases of all
    patterns, in every other column the negative of a product in the column, which leaves sums near zero."""
    rng = np.random.default_rng(M + K + up)
    A, B = (fast.round_from_float((rng.standard_normal(s) * 2.0 ** up).astype(np.float32), fmt) for s in ((M, K), (K, N)))
    bv = _operand(rng, (N,), fmt, "uniform")
    part, _ = fast.gemm(np.ascontiguousarray(A[:1]), B, fmt, fmt)
    bv[::2] = (-part[0, ::2].astype(np.int64)).astype(bv.dtype) & ((1 << BITS[fmt]) - 1)
    bv[5] = 1 << (BITS[fmt] - 1)
    got = to_np(pn.posit_gemm(to_dev(A), to_dev(B), fmt, fout, bias=to_dev(bv)), fout)
    rows = np.array([0, 1, 31, 32, 63, 64, 500, M - 2, M - 1])
    want, _ = fast.gemm(np.ascontiguousarray(A[rows]), B, fmt, fout, bias=bv)
    assert len(mismatches(got[rows], want)) == 0
    assert (got[:, 5] == 1 << (BITS[fout] - 1)).all()


@pytest.mark.parametrize("fmt", ["p8_1", "p8_2", "p16", "p12_1", "p32"])
@pytest.mark.parametrize("nar", [False, True])
def test_windows_at_their_limits(fmt, nar):
    """Magnitudes from lo up to hi = the largest span that a kernel takes, one pattern more, and one less, the extremes
    present in both operands."""
    M, N, K = 520, 512, 288
    rng = np.random.default_rng(BITS[fmt])
    one = 1 << (BITS[fmt] - 2)
    spans = [s * (1 << max(0, BITS[fmt] - 8)) for s in (6, 20, 40, 55, 61)]
    for span in spans:
        lo, hi = max(1, one - span), min((1 << (BITS[fmt] - 1)) - 1, one + span)
        ops = []
        for shape in ((M, K), (K, N)):
            m = rng.integers(lo, hi + 1, size=shape, dtype=np.int64)
            m.reshape(-1)[[0, -1]] = lo, hi
            x = np.where(rng.random(shape) < 0.5, m, (1 << BITS[fmt]) - m).astype(NP_DTYPE[fmt])
            ops.append(x)
        if nar:
            ops[0][5, 7] = 1 << (BITS[fmt] - 1)
        got = to_np(pn.posit_gemm(to_dev(ops[0]), to_dev(ops[1]), fmt, fmt), fmt)
        rows = np.array([0, 5, 6, 63, 64, M - 1])
        want, _ = fast.gemm(np.ascontiguousarray(ops[0][rows]), ops[1], fmt, fmt)
        assert len(mismatches(got[rows], want)) == 0, (fmt, span, nar)


def test_p8_1_narrow_kernel_and_its_neighbour():
    """2^31 products: the kernel of three planes, and (extremes present) the one of four behind it."""
    M, N, K = 1300, 1290, 1296
    for kinds in (("gauss", "relu"), ("uniform", "gauss")):
        _check("p8_1", "p8_1", M, N, K, 0, 1, kinds)


def test_static_scratch_gives_way_to_the_older_kernels():
    """posit_gemm_static takes what it took: where the digit planes exceed the fixed array, the older kernels serve."""
    M, N, K = 4096, 4100, 1280
    rng = np.random.default_rng(5)
    A, B = _operand(rng, (M, K), "p32", "gauss"), _operand(rng, (K, N), "p32", "gauss")
    assert pn.posit_gemm_workspace("p32", "p32", 0, 0, M, N, K) > 72 << 20
    got = to_np(pn.posit_gemm_static(to_dev(A), to_dev(B), "p32", "p32"), "p32")
    same = to_np(pn.posit_gemm(to_dev(A), to_dev(B), "p32", "p32"), "p32")
    assert np.array_equal(got, same)
    want, _ = fast.gemm(np.ascontiguousarray(A[[0, M - 1]]), B, "p32", "p32")
    assert np.array_equal(got[[0, M - 1]], want)


@pytest.mark.parametrize("fmt,fout,M,N,K,ta,tb", [("p16", "p16", 96, 97, 4097, 0, 1), ("p16", "p32", 130, 700, 1056, 1, 0), ("p16", "p8", 100, 97, 16352, 0, 0),
                                                  ("p12_1", "p12_1", 162, 210, 3956, 0, 1), ("p10_1", "p16", 121, 319, 2993, 1, 1)])
@pytest.mark.parametrize("bias,nar", [(False, False), (True, True)])
def test_wide_windows_cut_into_slices(fmt, fout, M, N, K, ta, tb, bias, nar):
    """Few tiles and a long reduction over operands that need all planes: the wide kernel's slices and their merge."""
    rng = np.random.default_rng(M + N + K)
    A, B = (rand_patterns(rng, s, fmt, special=0.01, allow_nar=False) for s in ((M, K), (K, N)))
    if nar:
        A[M - 1, K - 1] = A[3, 0] = B[K // 2, N - 1] = 1 << (BITS[fmt] - 1)
    bv = _operand(rng, (N,), fmt, "uniform") if bias else None
    Ain, Bin = (np.ascontiguousarray(A.T) if ta else A), (np.ascontiguousarray(B.T) if tb else B)
    got = to_np(pn.posit_gemm(to_dev(Ain), to_dev(Bin), fmt, fout, trans_a=ta, trans_b=tb, bias=None if bv is None else to_dev(bv)), fout)
    rows = np.array([0, 3, 31, 32, 63, 64, M - 1])
    want, _ = fast.gemm(np.ascontiguousarray(A[rows]), B, fmt, fout, bias=bv)
    bad = mismatches(got[rows], want)
    assert len(bad) == 0, "%d outputs differ, first at %s" % (len(bad), bad[0])


def test_posit32_with_bias_takes_no_workspace():
    import torch
    from paper_2105_00053_amd import binding
    M, N, K = 450, 470, 256
    rng = np.random.default_rng(32)
    A, B, bias = _operand(rng, (M, K), "p32", "gauss"), _operand(rng, (K, N), "p32", "gauss"), _operand(rng, (N,), "p32", "gauss")
    a, b, v, c = to_dev(A), to_dev(B), to_dev(bias), torch.zeros((M, N), dtype=torch.int32, device="cuda")
    code, stream = binding.FORMAT_CODES["p32"], torch.cuda.current_stream().cuda_stream
    call = binding.load().posit_gemm
    assert call(stream, code, code, 0, 0, M, N, K, a.data_ptr(), K, b.data_ptr(), N, v.data_ptr(), c.data_ptr(), N, None, 0) == 0
    want, _ = fast.gemm(A, B, "p32", "p32", bias=bias)
    assert len(mismatches(to_np(c, "p32"), want)) == 0
    assert call(stream, code, code, 0, 0, M, N, K, a.data_ptr(), K, b.data_ptr(), N, None, c.data_ptr(), N, None, 0) == 3


@pytest.mark.parametrize("fmt,M,N,K,ta,tb,bias,fout", [
    ("p16", 96, 96, 64, False, False, False, "p16"),       # two k blocks for four waves
    ("p12_1", 97, 129, 65, True, False, True, "p12_1"),    # one row, column and index into the last tile and block
    ("p10_1", 127, 96, 127, False, True, True, "p10_1"),   # four k blocks, the last one short
    ("p16", 160, 161, 161, True, True, True, "p32"),       # six k blocks: waves with one and with two; wide output
    ("p12_1", 300, 333, 991, False, False, False, "p8"),   # the longest reduction that is not cut: eight steps a wave
    ("p16", 1024, 448, 96, False, True, False, "p16"),     # the last number of tiles that goes here, and the first beyond
    ("p16", 1024, 449, 96, False, True, False, "p16"),
    ("p8_2", 256, 270, 500, True, False, True, "p12_2"),
    ("p8_1", 256, 1024, 1023, False, True, True, "p8_1"),  # one workgroup per compute unit
    ("p8_1", 640, 704, 500, True, False, False, "p12_1"),  # the longest reduction of that many tiles, and the first beyond
    ("p8_1", 640, 704, 501, False, False, True, "p8_1"),
])
def test_few_tiles_of_32_by_32(fmt, M, N, K, ta, tb, bias, fout):
    """The kernel whose waves share the reduction of one 32 x 32 tile: N(0, 1) operands with NaR in the first row, the last
    column and in the bias; also data over the whole range, which it leaves to the kernel of more planes."""
    rng = np.random.default_rng([23, M, N, K])
    for kind in ("normal", "wide"):
        A, B = (fast.round_from_float(rng.standard_normal(s).astype(np.float32), fmt) for s in ((M, K), (K, N)))
        if kind == "wide":
            A = rand_patterns(rng, (M, K), fmt, allow_nar=False)
        nar = NP_DTYPE[fmt](1 << (BITS[fmt] - 1))
        A[0, K - 1] = nar
        B[K // 2, N - 1] = nar
        b = None
        if bias:
            b = fast.round_from_float(rng.standard_normal(N).astype(np.float32), fmt)
            b[1] = nar
        C = pn.posit_gemm(to_dev(A.T if ta else A), to_dev(B.T if tb else B), fmt, fout, trans_a=ta, trans_b=tb, bias=None if b is None else to_dev(b))
        want, _ = fast.gemm(A, B, fmt, fout, bias=b)
        assert len(mismatches(to_np(C, fout), want)) == 0, kind
