"""GPU parity of the digit-plane convolutions that hold one pair of k blocks of 32 in LDS, reductions of one block to fourteen, against the C++ oracle, bit for
bit: both shapes of a workgroup, ragged positions, biases, NaR on either side, operands that four planes hold and that take the wide kernel."""
import ctypes

import numpy as np
import pytest

import paper_2105_00053_amd as pn
from oracle import fast

from gpu_util import BITS, mismatches, rand_patterns, to_dev, to_np
from test_host_logic import CODE, hc  # noqa: F401

pytestmark = pytest.mark.gpu

# gathered channels, outputs' channels, filter: 1, 1, 2, 2, 3, 2, 5, 9 and 14 k blocks
LAYERS = [(16, 40, 1), (30, 100, 1), (33, 24, 1), (64, 70, 1), (65, 40, 1), (7, 18, 2), (5, 20, 3), (20, 40, 3), (33, 24, 3)]


CASES = [(False, f, w, l) for f in ("p8_2", "p12_1", "p16") for w in (0, 1) for l in LAYERS] + [(True, "p10_1", w, l) for w in (0, 1) for l in LAYERS[:4:2] + LAYERS[7:8]]


@pytest.mark.parametrize("wide,fmt,which,layer", CASES)
def test_passes(hc, wide, fmt, which, layer):  # noqa: F811
    ci, mo, r = layer
    n, h = (70, 33) if r == 1 else (70, 36) if r == 2 else (52, 33)  # more than 768 workgroups
    c, k = (ci, mo) if which == 0 else (mo, ci)
    d = dict(N=n, C=c, H=h, W=h, K=k, R=r, S=r, pad_h=0, pad_w=0, stride_h=1, stride_w=1)
    desc = pn.ConvDesc(n, c, h, h, k, r, r, 0, 0, 1, 1)
    hc.hostcheck_conv_gather_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    hc.hostcheck_direct_conv_plan.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    assert hc.hostcheck_conv_gather_plan(CODE[fmt], which, ctypes.byref(desc), (ctypes.c_int64 * 12)())
    assert not hc.hostcheck_direct_conv_plan(CODE[fmt], which, ctypes.byref(desc), 0, (ctypes.c_int64 * 6)())
    rng = np.random.default_rng(ci + which)
    oh = h - r + 1
    nar, one = 1 << (BITS[fmt] - 1), 1 << (BITS[fmt] - 2)

    def tensor(*shape):
        if wide:
            return rand_patterns(rng, shape, fmt, special=0.02, allow_nar=False)
        p = fast.round_from_float(rng.standard_normal(shape).astype(np.float32), fmt)
        p[np.abs(p.astype(np.int64) - one) > one // 2] = one  # few bits: four planes hold them
        return p

    w = tensor(k, c, r, r)
    if which == 0:
        x, bias = tensor(n, c, h, h), tensor(k)
        x[n - 1, c - 1, h - 1, h - 1] = nar
        bias[0] = nar
        got, want = pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, fmt, bias=to_dev(bias)), fast.conv2d_fwd(x, w, d, fmt, fmt, bias=bias)
        assert len(mismatches(to_np(got, fmt), want)) == 0
        w[k - 1, 0, 0, 0] = nar
        got, want = pn.posit_conv2d_fwd(to_dev(x), to_dev(w), desc, fmt, "p32"), fast.conv2d_fwd(x, w, d, fmt, "p32")
        assert len(mismatches(to_np(got, "p32"), want)) == 0
    else:
        dy = tensor(n, k, oh, oh)
        dy[0, 0, 0, 0] = w[0, c - 1, 0, 0] = nar
        for fout in (fmt, "p32"):
            got, want = pn.posit_conv2d_bwd_data(to_dev(dy), to_dev(w), desc, fmt, fout), fast.conv2d_bwd_data(dy, w, d, fmt, fout)
            assert len(mismatches(to_np(got, fout), want)) == 0
