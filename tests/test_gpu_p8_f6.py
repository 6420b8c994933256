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


def _digits():
    """h and l of every pattern."""
    L = ctypes.CDLL(build.HOSTCHECK)
    out, h, l = np.zeros(6, dtype=np.int32), np.zeros(256, dtype=np.int64), np.zeros(256, dtype=np.int64)
    for p in range(256):
        L.hostcheck_p8_f6(ctypes.c_uint32(p), out.ctypes.data_as(ctypes.c_void_p))
        h[p], l[p] = out[1:3]
    return h, l


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
    if kind == "one sign":  # every product positive: the largest sums of such data
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


LIMIT = 16776000.0  # of the low sum's bound; the bound of the high one is a sixteenth


def _bounds(A, B):
    """The bounds the kernel works out: of the high sum and of the low one."""
    h, l = _digits()
    norms = [[np.sqrt(np.add.reduceat(d[X] ** 2, np.arange(0, X.shape[1], 256), axis=1).max(axis=0).astype(np.float64)) for d in (h, l)] for X in (A, B.T)]
    (ha, la), (hb, lb) = norms
    return (ha * hb).sum(), (32 * (ha * lb + la * hb) + la * lb).sum()


def _at_the_bound(K):
    """24 (h = 48) against 15/64 (l = 15): Cauchy's inequality is an equality, so the low sum itself comes up to the bound, in steps of
    one unit (rows with 1/64 in places).  Every other row is negative; in half of the columns eight large entries bring the high
    sum against it, to about three, so that its rounding sees the low units."""
    rng = np.random.default_rng(11)
    A, B = np.full((2048, K), 0x7D, np.uint8), np.full((K, 2048), 0x0F, np.uint8)
    A[1::2] = 0x83
    A[2::4][rng.random((512, K)) < 0.003] = 0x01
    A[3::4][rng.random((512, K)) < 0.003] = 0xFF
    for n in range(1, 2048, 2):
        B[rng.choice(K, n // 2 % 7, replace=False), n] = 0x0E
    large = np.array([0x83] * 6 + [0x84] + [0x100 - 0x76], np.uint8)  # -24, -16, -7
    for n in range(2, 2048, 4):
        B[rng.choice(K, 8, replace=False), n] = large
        B[rng.choice(K, 8, replace=False), n + 1] = large
    return A, B


@pytest.mark.gpu
@pytest.mark.parametrize("fout", ["p8", "p32"])
def test_sums_at_the_bound_are_exact(fout):
    A, B = _at_the_bound(720)
    bhh, bq = _bounds(A, B)
    assert bhh < LIMIT / 16 and 0.98 * 2 ** 24 < bq < LIMIT
    rows = np.concatenate([np.arange(8), np.arange(1020, 1036)])
    h, l = _digits()
    ha, la, hb, lb = (X.astype(np.float64) for X in (h[A[rows]], l[A[rows]], h[B], l[B]))  # exact: integers far below 2^53
    q = 32 * (ha @ lb + la @ hb) + la @ lb
    assert np.abs(q).max() > 0.98 * 2 ** 24 and len(np.unique(q % 1536)) > 20  # at the bound, and not in steps of a cross product
    workspace = torch.empty(pn.posit_gemm_workspace("p8", fout, False, False, 2048, 2048, 720), dtype=torch.uint8, device="cuda")
    C = pn.posit_gemm(to_dev(A), to_dev(B), "p8", fout, workspace=workspace)
    assert workspace[-4:].tolist() == [0x80] * 4  # the 6-bit kernel's verdict: done there
    want, _ = fast.gemm(np.ascontiguousarray(A[rows]), B, "p8", fout)
    assert len(np.unique(want.reshape(len(rows), -1, 4)[:, :, 2:])) > 20  # no saturation where the sums cancel
    assert len(mismatches(to_np(C, fout)[rows], want)) == 0


@pytest.mark.gpu
def test_captured_product_follows_the_data_of_each_replay():
    """One captured call on one workspace, its operands changed between replays: taken in 6 bits, refused by a value without digits,
    by the bound, and taken again."""
    M, N, K = 2176, 2050, 700
    kinds = ["normal", "special", "normal", "large", "patterns", "normal"]
    sets = [_operands(kind, M, N, K) for kind in kinds]
    A, B = (to_dev(x) for x in sets[0])
    out = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    workspace = torch.empty(pn.posit_gemm_workspace("p8", "p8", False, False, M, N, K), dtype=torch.uint8, device="cuda")
    pn.posit_gemm(A, B, "p8", "p8", out=out, workspace=workspace)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pn.posit_gemm(A, B, "p8", "p8", out=out, workspace=workspace)
    rows = np.concatenate([np.arange(4), np.arange(128, 132), [300], np.arange(M - 3, M)])
    for kind, (a, b) in zip(kinds, sets):
        A.copy_(to_dev(a))
        B.copy_(to_dev(b))
        out.fill_(0x55)
        graph.replay()
        torch.cuda.synchronize()
        assert (workspace[-4:].tolist() == [0x80] * 4) == (kind == "normal")
        want, _ = fast.gemm(np.ascontiguousarray(a[rows]), b, "p8", "p8")
        assert len(mismatches(to_np(out, "p8")[rows], want)) == 0, kind
        assert torch.equal(out, pn.posit_gemm(A, B, "p8", "p8")), kind


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
