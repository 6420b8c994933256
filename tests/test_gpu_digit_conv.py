"""The three convolution passes of posit(8,1), (8,2), (10,1), (12,1) and <16,1> on the integer matrix cores: geometries at
the edges of tiles, channel groups and image groups, strides, paddings up to the filter and beyond, 3 to 70 output channels
(both tile shapes), windows that four planes hold and ones that need eight, NaR, the bias and its gradient, and a
weight gradient whose quire wraps.  Bit-exact against the oracle."""
import numpy as np
import pytest

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, NP_DTYPE, mismatches, rand_patterns, to_dev, to_np

pytestmark = pytest.mark.gpu
MASTER = {"p8": "p16", "p8_1": "p12_1", "p8_2": "p12_2", "p10_1": "p10_1", "p12_1": "p8_2", "p16": "p16"}

GEOMETRIES = [
    dict(N=33, C=17, H=15, W=13, K=33, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=16, C=16, H=20, W=20, K=32, R=1, S=1, pad_h=0, pad_w=0),
    dict(N=50, C=3, H=17, W=19, K=31, R=5, S=4, pad_h=2, pad_w=4),
    dict(N=20, C=40, H=12, W=14, K=70, R=2, S=3, pad_h=0, pad_w=0),
    dict(N=15, C=20, H=25, W=24, K=64, R=3, S=3, pad_h=1, pad_w=1, stride_h=2, stride_w=1),
    dict(N=64, C=6, H=14, W=14, K=16, R=5, S=5, pad_h=0, pad_w=0),
    dict(N=17, C=48, H=16, W=16, K=3, R=3, S=3, pad_h=3, pad_w=2),
    dict(N=40, C=33, H=17, W=16, K=31, R=3, S=3, pad_h=1, pad_w=1),
    dict(N=67, C=40, H=16, W=16, K=3, R=5, S=5, pad_h=2, pad_w=2),
    dict(N=21, C=16, H=20, W=20, K=32, R=1, S=1, pad_h=0, pad_w=0),
    dict(N=2, C=30, H=50, W=52, K=40, R=3, S=3, pad_h=1, pad_w=1),
]


def _desc(d):
    full = dict(stride_h=1, stride_w=1)
    full.update(d)
    return pn.ConvDesc(full["N"], full["C"], full["H"], full["W"], full["K"], full["R"], full["S"], full["pad_h"], full["pad_w"], full["stride_h"],
                       full["stride_w"])


def _tensor(rng, shape, fmt, kind, sigma=1.0):
    if kind == "uniform":
        return rand_patterns(rng, shape, fmt, special=0.001, allow_nar=False)
    return fast.round_from_float((rng.standard_normal(shape) * sigma).astype(np.float32), fmt)


def _equal(got, want, what):
    bad = mismatches(got, want)
    assert len(bad) == 0, "%s: %d of %d outputs differ, first at %s" % (what, len(bad), want.size, bad[0])


@pytest.mark.parametrize("geometry", range(len(GEOMETRIES)))
@pytest.mark.parametrize("kind", ["gauss", "uniform"])
@pytest.mark.parametrize("fmt", ["p8_1", "p8_2", "p10_1", "p12_1", "p16"])
def test_three_passes(fmt, kind, geometry):
    d = GEOMETRIES[geometry]
    rng = np.random.default_rng(geometry + BITS[fmt])
    nar, fm, desc = 1 << (BITS[fmt] - 1), MASTER[fmt], _desc(d)
    oh, ow = fast.out_hw(d)
    x = np.maximum(0, _tensor(rng, (d["N"], d["C"], d["H"], d["W"]), fmt, kind)) if kind == "uniform" else _tensor(rng, (d["N"], d["C"], d["H"], d["W"]), fmt, kind)
    w = _tensor(rng, (d["K"], d["C"], d["R"], d["S"]), fmt, kind, 0.1)
    dy = _tensor(rng, (d["N"], d["K"], oh, ow), fmt, kind, 1 / 64)
    bias = _tensor(rng, (d["K"],), fmt, "uniform")
    bias[d["K"] - 1] = nar
    x[0, d["C"] - 1, d["H"] // 2, d["W"] // 2] = nar
    w[1, 0, d["R"] - 1, 0] = nar
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, fmt, bias=to_dev(bias)), fmt)
    _equal(y, fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias), "forward with bias")
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, "p32"), "p32")
    _equal(y, fast.conv2d_fwd(x, w, d, fmt, "p32"), "forward to posit<32,2>")
    dy[d["N"] - 1, 0, 0, ow - 1] = nar
    dx = to_np(pn.posit_conv2d_bwd_data(to_dev(dy), to_dev(w), desc, fmt, fmt), fmt)
    _equal(dx, fast.conv2d_bwd_data(dy, w, d, fmt, fmt), "backward-data")
    dw, db = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), desc, fmt, fm, with_bias=True)
    wdw, wdb = fast.conv2d_bwd_weight(dy, x, d, fmt, fm, with_bias=True)
    _equal(to_np(dw, fm), wdw, "backward-weight")
    _equal(to_np(db, fm), wdb, "bias gradient")
    only = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), desc, fmt, fmt)
    _equal(to_np(only[0] if isinstance(only, tuple) else only, fmt), fast.conv2d_bwd_weight(dy, x, d, fmt, fmt), "backward-weight without bias gradient")


@pytest.mark.parametrize("pad", [16384, 16385, 40000, 49152])
@pytest.mark.parametrize("fmt", ["p8_1", "p8_2", "p12_1", "p16"])
def test_paddings_beyond_the_tensor(fmt, pad):
    """Paddings of thousands of rows under a stride that lands one output row on the tensor: beyond 16 bits of offset the
    general kernel serves."""
    d = dict(N=64, C=16, H=7, W=9, K=128, R=3, S=3, pad_h=pad, pad_w=1, stride_h=pad // 2, stride_w=1)
    rng = np.random.default_rng(pad + BITS[fmt])
    x, w, dy = _tensor(rng, (64, 16, 7, 9), fmt, "gauss"), _tensor(rng, (128, 16, 3, 3), fmt, "gauss"), _tensor(rng, (64, 128) + fast.out_hw(d), fmt, "gauss")
    bias = _tensor(rng, (128,), fmt, "gauss")
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), _desc(d), fmt, fmt, bias=to_dev(bias)), fmt)
    _equal(y, fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias), "forward")
    assert len(np.unique(y[:, 0])) > 8  # some output row reads the tensor
    dw, db = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), _desc(d), fmt, fmt, with_bias=True)
    wdw, wdb = fast.conv2d_bwd_weight(dy, x, d, fmt, fmt, with_bias=True)
    _equal(to_np(dw, fmt), wdw, "backward-weight")
    _equal(to_np(db, fmt), wdb, "bias gradient")


@pytest.mark.parametrize("pad", [16384, 16385, 40000, 65534])
def test_paddings_beyond_the_tensor_posit8_0(pad):
    """The same for posit<8,0>, whose matrix-core kernels serve stride 1 only."""
    d = dict(N=1, C=16, H=40, W=1, K=32, R=3, S=1, pad_h=pad, pad_w=0)
    rng = np.random.default_rng(pad)
    x, w = _tensor(rng, (1, 16, 40, 1), "p8", "gauss"), _tensor(rng, (32, 16, 3, 1), "p8", "gauss")
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), _desc(d), "p8", "p8"), "p8")
    _equal(y, fast.conv2d_fwd(x, w, d, "p8", "p8"), "forward")
    assert len(np.unique(y)) > 32


@pytest.mark.parametrize("C,N,H,K", [(512, 37, 15, 5), (514, 43, 14, 5), (528, 37, 15, 5), (4096, 43, 14, 5), (4100, 43, 14, 64), (4100, 43, 14, 65),
                                     (8192, 37, 15, 70)])
def test_many_channels_posit8_0(C, N, H, K):
    """Up to 32 groups of 16 input channels a workgroup writes the digits of a stretch of pixels, beyond of one group; 512 groups
    are the most the kernel takes, beyond 256 with more than 64 outputs only."""
    d = dict(N=N, C=C, H=H, W=H, K=K, R=1, S=1, pad_h=0, pad_w=0)
    rng = np.random.default_rng(C + H)
    x, w, bias = _tensor(rng, (N, C, H, H), "p8", "gauss"), _tensor(rng, (K, C, 1, 1), "p8", "gauss", 0.1), _tensor(rng, (K,), "p8", "gauss")
    x[N - 1, C - 1, H - 1, H - 1] = 0x80
    w[3, C - 2] = 0x80
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), _desc(d), "p8", "p8", bias=to_dev(bias)), "p8")
    images = np.array([0, N // 2, N - 1])
    _equal(y[images], fast.conv2d_fwd(np.ascontiguousarray(x[images]), w, dict(d, N=3), "p8", "p8", bias=bias), "forward")


@pytest.mark.parametrize("spans", [(22, 34), (34, 22), (38, 30), (30, 46), (46, 38), (46, 46), (56, 22)])
@pytest.mark.parametrize("fmt,maxs", [("p8_2", 24), ("p10_1", 16), ("p12_1", 20), ("p16", 28)])
def test_planes_that_hold_anything(fmt, maxs, spans):
    """Operands whose values span so many powers of two: the wide kernel multiplies four to seven planes of each, or all
    eight, without NaR; the spans lie at the bottom, in the middle and at the top of the format's range."""
    d = GEOMETRIES[0 if spans[0] < 40 else 6]
    desc, fm = _desc(d), MASTER[fmt]
    oh, ow = fast.out_hw(d)
    rng = np.random.default_rng(spans[0] * 64 + spans[1])

    def tensor(shape, span, at):
        low = -maxs + at * (2 * maxs - min(span, 2 * maxs))
        v = np.exp2(low + rng.random(shape) * min(span, 2 * maxs)) * rng.choice([-1.0, 1.0], size=shape)
        return fast.round_from_float(v.astype(np.float32), fmt)

    x, w, dy = tensor((d["N"], d["C"], d["H"], d["W"]), spans[0], 0), tensor((d["K"], d["C"], d["R"], d["S"]), spans[1], 1), tensor((d["N"], d["K"], oh, ow), spans[1], 0.5)
    bias = tensor((d["K"],), 2 * maxs, 0)
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, fmt, bias=to_dev(bias)), fmt)
    _equal(y, fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias), "forward")
    dx = to_np(pn.posit_conv2d_bwd_data(to_dev(dy), to_dev(w), desc, fmt, fmt), fmt)
    _equal(dx, fast.conv2d_bwd_data(dy, w, d, fmt, fmt), "backward-data")
    dw, db = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), desc, fmt, fm, with_bias=True)
    wdw, wdb = fast.conv2d_bwd_weight(dy, x, d, fmt, fm, with_bias=True)
    _equal(to_np(dw, fm), wdw, "backward-weight")
    _equal(to_np(db, fm), wdb, "bias gradient")


@pytest.mark.parametrize("fmt,C,K", [("p8", 64, 6), ("p8", 64, 33), ("p8_1", 128, 4), ("p8_2", 64, 33), ("p10_1", 128, 4), ("p12_1", 128, 4), ("p16", 64, 33), ("p16", 128, 4)])
def test_weight_gradient_with_whole_column_tiles(fmt, C, K):
    """C R S a multiple of the column tile (64, or 128 for at most 32 output channels): without the bias column the product has
    a tile less and the reduction more slices."""
    d = dict(N=16, C=C, H=31, W=31, K=K, R=3, S=3, pad_h=1, pad_w=1)
    rng = np.random.default_rng(C + K + BITS[fmt])
    x, dy = _tensor(rng, (16, C, 31, 31), fmt, "gauss"), _tensor(rng, (16, K, 31, 31), fmt, "gauss", 1 / 16)
    want, wdb = fast.conv2d_bwd_weight(dy, x, d, fmt, MASTER[fmt], with_bias=True)
    only = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), _desc(d), fmt, MASTER[fmt])
    _equal(to_np(only[0] if isinstance(only, tuple) else only, MASTER[fmt]), want, "backward-weight without bias gradient")
    dw, db = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), _desc(d), fmt, MASTER[fmt], with_bias=True)
    _equal(to_np(dw, MASTER[fmt]), want, "backward-weight")
    _equal(to_np(db, MASTER[fmt]), wdb, "bias gradient")


@pytest.mark.parametrize("fmt", ["p8_1", "p16", "p12_1"])
def test_weight_gradient_wraps_like_the_quire(fmt):
    """45056 products of maxpos leave a quire that guarantees 32767: it wraps modulo 2^bits, in the oracle and here."""
    d = dict(N=44, C=8, H=32, W=32, K=20, R=1, S=1, pad_h=0, pad_w=0)
    maxpos = (1 << (BITS[fmt] - 1)) - 1
    x = np.full((d["N"], d["C"], d["H"], d["W"]), maxpos, dtype=NP_DTYPE[fmt])
    dy = np.full((d["N"], d["K"], d["H"], d["W"]), maxpos, dtype=NP_DTYPE[fmt])
    dy[:, 1] = 1 << (BITS[fmt] - 2)  # ones: this channel does not wrap
    dy[3, 2] = 0
    dw = to_np(pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), _desc(d), fmt, fmt), fmt)
    want = fast.conv2d_bwd_weight(dy, x, d, fmt, fmt)
    _equal(dw, want, "wrapped weight gradient")
    assert dw[0, 0, 0, 0] >= 1 << (BITS[fmt] - 1) and dw[1, 0, 0, 0] < 1 << (BITS[fmt] - 1)  # negative, positive


def test_captured_calls_follow_the_data():
    """The kernel that serves is chosen on the device: a captured forward and weight gradient replayed on operands that four
    planes hold, ones that need eight, and the first kind again, with a workspace full of ones."""
    import torch
    fmt, d = "p16", dict(N=20, C=16, H=18, W=18, K=24, R=3, S=3, pad_h=1, pad_w=1)
    desc = _desc(d)
    rng = np.random.default_rng(4)
    xs, ws, dys = (torch.zeros(s, dtype=torch.int16, device="cuda") for s in ((20, 16, 18, 18), (24, 16, 3, 3), (20, 24, 18, 18)))
    y, dw = torch.zeros((20, 24, 18, 18), dtype=torch.int16, device="cuda"), torch.zeros((24, 16, 3, 3), dtype=torch.int16, device="cuda")
    need = max(pn.posit_conv2d_workspace(k, fmt, fmt, desc) for k in (0, 2))
    scratch = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")

    def calls():
        pn.posit_conv2d_fwd(xs, ws, desc, fmt, fmt, out=y, workspace=scratch)
        pn.posit_conv2d_bwd_weight(dys, xs, desc, fmt, fmt, out=dw, workspace=scratch)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for kind in ("gauss", "uniform", "gauss", "gauss"):
        x, w, dy = (_tensor(rng, tuple(t.shape), fmt, kind) for t in (xs, ws, dys))
        for t, v in ((xs, x), (ws, w), (dys, dy)):
            t.copy_(to_dev(v))
        y.fill_(0x55)
        dw.fill_(0x55)
        graph.replay()
        torch.cuda.synchronize()
        _equal(to_np(y, fmt), fast.conv2d_fwd(x, w, d, fmt, fmt), "replayed forward, " + kind)
        _equal(to_np(dw, fmt), fast.conv2d_bwd_weight(dy, x, d, fmt, fmt), "replayed weight gradient, " + kind)
