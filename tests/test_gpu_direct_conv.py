"""Small layers on the matrix cores straight from their patterns (direct_mfma.h, direct_conv.hip), the three passes against the C++
oracle, bit for bit: rows, columns and reductions around the tiles, the k blocks and the slices, strides in every pass, paddings beyond the filter, one
channel, one position, every format, NaR, biases and their gradient."""
import numpy as np
import pytest
import torch

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, mismatches, rand_patterns, to_dev, to_np

pytestmark = pytest.mark.gpu
MASTER = {"p8": "p16", "p8_1": "p12_1", "p8_2": "p12_2", "p10_1": "p10_1", "p10_2": "p12_2", "p12_1": "p8_2", "p12_2": "p12_2", "p16": "p16"}

GEOMETRIES = [  # N, C, H, W, K, R, S, pad_h, pad_w, stride_h, stride_w
    (3, 1, 28, 28, 6, 5, 5, 2, 2, 1, 1),
    (5, 6, 14, 13, 16, 5, 5, 0, 0, 1, 1),
    (7, 17, 9, 11, 33, 3, 2, 1, 1, 2, 3),
    (2, 16, 16, 16, 15, 1, 1, 0, 0, 2, 2),
    (1, 3, 7, 9, 5, 7, 9, 0, 0, 1, 1),
    (9, 8, 5, 6, 17, 3, 3, 4, 3, 1, 2),
    (31, 12, 8, 8, 31, 3, 3, 1, 1, 1, 1),
    (4, 65, 6, 5, 64, 2, 4, 1, 3, 2, 1),
    (16, 2, 12, 12, 1, 4, 4, 0, 0, 4, 4),
]


def _equal(got, want, what):
    bad = mismatches(got, want)
    assert len(bad) == 0, "%s: %d of %d outputs differ, first at %s" % (what, len(bad), want.size, bad[0])


def _three_passes(fmt, geometry, nar, seed):
    rng = np.random.default_rng(seed)
    d = dict(zip(("N", "C", "H", "W", "K", "R", "S", "pad_h", "pad_w", "stride_h", "stride_w"), geometry))
    desc, fm, mark = pn.ConvDesc(*geometry), MASTER[fmt], 1 << (BITS[fmt] - 1)
    oh, ow = fast.out_hw(d)
    tensor = lambda *shape: rand_patterns(rng, shape, fmt, special=0.05, allow_nar=False)
    x, w, dy, bias = tensor(d["N"], d["C"], d["H"], d["W"]), tensor(d["K"], d["C"], d["R"], d["S"]), tensor(d["N"], d["K"], oh, ow), tensor(d["K"])
    if nar:
        bias[-1] = mark
        x[0, d["C"] - 1, d["H"] // 2, d["W"] // 2] = mark
        w[d["K"] // 2, 0, d["R"] - 1, 0] = mark
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, fmt, bias=to_dev(bias)), fmt)
    _equal(y, fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias), "forward with bias")
    y = to_np(pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, "p32"), "p32")
    _equal(y, fast.conv2d_fwd(x, w, d, fmt, "p32"), "forward to posit<32,2>")
    if nar:
        dy[-1, 0, 0, ow - 1] = mark
    dx = to_np(pn.posit_conv2d_bwd_data(to_dev(dy), to_dev(w), desc, fmt, fmt), fmt)
    _equal(dx, fast.conv2d_bwd_data(dy, w, d, fmt, fmt), "backward-data")
    dw, db = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), desc, fmt, fm, with_bias=True)
    wdw, wdb = fast.conv2d_bwd_weight(dy, x, d, fmt, fm, with_bias=True)
    _equal(to_np(dw, fm), wdw, "backward-weight")
    _equal(to_np(db, fm), wdb, "bias gradient")
    only = pn.posit_conv2d_bwd_weight(to_dev(dy), to_dev(x), desc, fmt, fmt)
    _equal(to_np(only[0] if isinstance(only, tuple) else only, fmt), fast.conv2d_bwd_weight(dy, x, d, fmt, fmt), "backward-weight without bias gradient")


@pytest.mark.parametrize("geometry", range(len(GEOMETRIES)))
@pytest.mark.parametrize("fmt", sorted(MASTER))
def test_three_passes(fmt, geometry):
    _three_passes(fmt, GEOMETRIES[geometry], geometry % 3 != 2, geometry)


@pytest.mark.parametrize("fmt", sorted(MASTER))
def test_long_reductions_in_slices(fmt):
    """Weight gradients over thousands of positions, the last slice a remainder."""
    _three_passes(fmt, (25, 5, 18, 17, 20, 3, 3, 1, 1, 1, 1), True, 3)


@pytest.mark.parametrize("fmt", ["p8", "p8_2", "p16"])
def test_less_workspace_than_asked_for(fmt):
    """A weight gradient whose workspace is smaller than the query says is refused or taken by another kernel, never run past its end."""
    import ctypes
    rng = np.random.default_rng(5)
    L, code, geometry = pn.load(), pn.binding.FORMAT_CODES[fmt], (25, 5, 18, 17, 20, 3, 3, 1, 1, 1, 1)
    desc = pn.ConvDesc(*geometry)
    need = L.posit_conv2d_workspace(2, code, code, ctypes.byref(desc))
    assert need > 0
    x, dy = rand_patterns(rng, (25, 5, 18, 17), fmt, allow_nar=False), rand_patterns(rng, (25, 20, 18, 17), fmt, allow_nar=False)
    xd, dyd = to_dev(x), to_dev(dy)
    dw = torch.zeros((20, 5, 3, 3), dtype=xd.dtype, device="cuda")
    stream, ptr = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), lambda t: ctypes.c_void_p(t.data_ptr())
    d = dict(zip(("N", "C", "H", "W", "K", "R", "S", "pad_h", "pad_w", "stride_h", "stride_w"), geometry))
    want = fast.conv2d_bwd_weight(dy, x, d, fmt, fmt)
    for given in (0, 16, need // 2 // 16 * 16, need - 1, need):
        ws = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        rc = L.posit_conv2d_bwd_weight(stream, code, code, ctypes.byref(desc), ptr(dyd), ptr(xd), ptr(dw), None, ptr(ws) if given else None, given)
        assert rc in (0, 3) and (given < need or rc == 0)
        assert bool((ws[given:] == 0xA5).all())
        if rc == 0:
            _equal(to_np(dw, fmt), want, "%d bytes" % given)
