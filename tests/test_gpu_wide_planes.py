"""Products and convolutions on four to eight digit planes, of sizes that go to these kernels, against the C++ oracle, bit for bit: edges of the tiles, odd and even numbers of k blocks, k blocks of which a few reach the lowest planes, slices, NaR, biases."""
import numpy as np
import pytest

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, mismatches, rand_patterns, to_dev, to_np

pytestmark = pytest.mark.gpu

# 63 / 64 / 65 and 31 / 32 / 33 beyond whole tiles; k blocks odd and even, a remainder of one index; few tiles and a long reduction
SIZES = [(959, 1055, 992), (960, 1024, 1025), (961, 1025, 1120), (897, 991, 1311), (130, 200, 16001)]


CASES = [(f, k) for f in ("p8_2", "p10_1", "p12_1", "p16") for k in ("window", "few", "many", "all")] + [("p32", "window")]


def _patterns(rng, shape, fmt, kind):
    a = fast.round_from_float(rng.standard_normal(shape).astype(np.float32), fmt)
    low, high = 1, (1 << (BITS[fmt] - 1)) - 1
    if kind == "all":
        return rand_patterns(rng, shape, fmt, allow_nar=False)
    n = {"few": 3, "many": a.size // 50, "window": 0}[kind]
    at = rng.integers(a.size, size=n)
    a.reshape(-1)[at] = np.where(np.arange(n) % 2, low, high).astype(a.dtype)
    return a


@pytest.mark.parametrize("fmt,kind", CASES)
@pytest.mark.parametrize("size", SIZES)
def test_product(fmt, kind, size):
    M, N, K = size
    rng = np.random.default_rng(M + len(kind))
    ta, tb = bool(M & 1), bool(N & 1)
    A, B = _patterns(rng, (K, M) if ta else (M, K), fmt, kind), _patterns(rng, (N, K) if tb else (K, N), fmt, kind)
    bias = rand_patterns(rng, (N,), fmt, special=0.1) if fmt != "p32" and kind != "few" else None
    if kind == "many":
        A[A.shape[0] // 2, 5] = B[3, B.shape[1] - 1] = 1 << (BITS[fmt] - 1)
    rows = np.unique(np.concatenate([[0, 5, 15, 16, 63, 64, M // 2, M - 1], rng.integers(M, size=6)]))
    opA = np.ascontiguousarray((A.T if ta else A)[rows])
    want, _ = fast.gemm(opA, B, fmt, fmt, trans_b=tb, bias=bias)
    got = to_np(pn.posit_gemm(to_dev(A), to_dev(B), fmt, fmt, trans_a=ta, trans_b=tb, bias=None if bias is None else to_dev(bias)), fmt)
    assert len(mismatches(got[rows], want)) == 0


# both tile shapes; pairs of k blocks whole (14) and with one left (25, 9), channels and positions beyond whole tiles, strides
LAYERS = [dict(N=64, C=48, H=16, W=16, K=70, R=3, S=3, pad_h=1, pad_w=1), dict(N=65, C=40, H=17, W=15, K=31, R=3, S=3, pad_h=1, pad_w=1),
          dict(N=40, C=32, H=18, W=18, K=33, R=5, S=5, pad_h=2, pad_w=2), dict(N=81, C=31, H=37, W=36, K=65, R=3, S=3, pad_h=0, pad_w=1, stride_h=2, stride_w=1)]


@pytest.mark.parametrize("fmt", ["p8_1", "p8_2", "p12_1", "p16"])
@pytest.mark.parametrize("kind", ["window", "many"])
@pytest.mark.parametrize("layer", range(len(LAYERS)))
def test_convolution(fmt, kind, layer):
    d = dict(stride_h=1, stride_w=1, **LAYERS[layer]) if "stride_h" not in LAYERS[layer] else LAYERS[layer]
    rng = np.random.default_rng(layer)
    desc = pn.ConvDesc(*(d[k] for k in ("N", "C", "H", "W", "K", "R", "S", "pad_h", "pad_w", "stride_h", "stride_w")))
    nar, (oh, ow) = 1 << (BITS[fmt] - 1), fast.out_hw(d)
    x, w = _patterns(rng, (d["N"], d["C"], d["H"], d["W"]), fmt, kind), _patterns(rng, (d["K"], d["C"], d["R"], d["S"]), fmt, kind)
    dy, bias = _patterns(rng, (d["N"], d["K"], oh, ow), fmt, kind), rand_patterns(rng, (d["K"],), fmt, special=0.1)
    if layer != 1:
        x[3, d["C"] - 1, 2, d["W"] - 1] = w[d["K"] - 1, 0, 0, 0] = dy[d["N"] - 1, 1, oh - 1, 0] = nar
    xd, wd, dyd = to_dev(x), to_dev(w), to_dev(dy)
    y = to_np(pn.posit_conv2d_fwd(xd, wd, desc, fmt, fmt, bias=to_dev(bias)), fmt)
    assert len(mismatches(y, fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias))) == 0
    assert len(mismatches(to_np(pn.posit_conv2d_fwd(xd, wd, desc, fmt, "p32"), "p32"), fast.conv2d_fwd(x, w, d, fmt, "p32"))) == 0
    assert len(mismatches(to_np(pn.posit_conv2d_bwd_data(dyd, wd, desc, fmt, fmt), fmt), fast.conv2d_bwd_data(dy, w, d, fmt, fmt))) == 0
    dw, db = pn.posit_conv2d_bwd_weight(dyd, xd, desc, fmt, fmt, with_bias=True)
    want = fast.conv2d_bwd_weight(dy, x, d, fmt, fmt, with_bias=True)
    assert len(mismatches(to_np(dw, fmt), want[0])) == 0 and len(mismatches(to_np(db, fmt), want[1])) == 0


@pytest.mark.parametrize("size", [(513, 511, 2049), (512, 1024, 1030), (130, 1030, 4000), (1024, 1023, 513), (353, 353, 5000)])
@pytest.mark.parametrize("order", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_posit8_0_few_tiles(size, order):
    """posit<8,0> on 128 to 1024 tiles of 32 x 32: edges of tiles, k blocks that do not divide by the waves, NaR, biases, output formats."""
    M, N, K = size
    ta, tb = map(bool, order)
    rng = np.random.default_rng(K)
    A, B = rand_patterns(rng, (K, M) if ta else (M, K), "p8", allow_nar=False), rand_patterns(rng, (N, K) if tb else (K, N), "p8", allow_nar=False)
    bias = rand_patterns(rng, (N,), "p8", special=0.1) if order != (0, 0) else None
    A[(K - 1, 3) if ta else (3, K - 1)] = B[(N - 1, K // 2) if tb else (K // 2, N - 1)] = 0x80
    for fout in ("p8", "p16", "p32"):
        got = to_np(pn.posit_gemm(to_dev(A), to_dev(B), "p8", fout, trans_a=ta, trans_b=tb, bias=None if bias is None else to_dev(bias)), fout)
        want, _ = fast.gemm(A, B, "p8", fout, trans_a=ta, trans_b=tb, bias=bias)
        assert len(mismatches(got, want)) == 0, fout
