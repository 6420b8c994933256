"""Which calls a training step makes, without a GPU: the binding is replaced by one that notes the calls."""
import types

import pytest
import torch

from paper_2105_00053_amd import train_step


def _calls(monkeypatch, fmt, n, cin, cout):
    seen = []
    empty = lambda *shape: torch.zeros(shape, dtype=torch.uint8)  # noqa: E731

    def gemm(a, b, fin, fout, trans_a=False, **_):
        seen.append("gemm")
        return empty(a.shape[1] if trans_a else a.shape[0], b.shape[1])

    def bwd_weight(dy, x, desc, fin, fout, with_bias):
        seen.append("bwd_weight")
        return empty(desc.K, desc.C, 1, 1), empty(desc.K)

    desc = lambda *v: types.SimpleNamespace(C=v[1], K=v[4])  # noqa: E731
    monkeypatch.setattr(train_step, "pn", types.SimpleNamespace(posit_gemm=gemm, posit_conv2d_bwd_weight=bwd_weight, ConvDesc=desc, posit_axpy_multi=lambda *a, **k: None))
    net = types.SimpleNamespace(compute=fmt, master=fmt, alpha=1, one=64, w16=[0], w8=[empty(cout, cin)], b16=[0], b8=[0])
    train_step.backward_and_update(net, [("fc", 0, None, empty(n, cin))], empty(n, cout))
    return seen


@pytest.mark.parametrize("fmt,n,cin,cout,joint", [("p8", 64, 400, 120, True), ("p16", 64, 84, 10, True), ("p8_2", 64, 400, 120, True), ("p32", 64, 400, 120, False),
                                                  ("p32", 1, 8, 2, False), ("p8", 500, 1537, 1000, False)])
def test_weight_gradient_of_a_fully_connected_layer(monkeypatch, fmt, n, cin, cout, joint):
    assert _calls(monkeypatch, fmt, n, cin, cout) == (["bwd_weight", "gemm"] if joint else ["gemm"] * 3)
