"""The C++ marshalling of the binding against the Python code it stands in for: the same outputs bit for bit (types, shapes,
given outputs), and the same errors, which the native code leaves to the Python code."""
import threading
import time

import pytest
import torch

import paper_2105_00053_amd as pn
from paper_2105_00053_amd import binding

pytestmark = pytest.mark.gpu


def _patterns(shape, fmt="p8", seed=1):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return pn.posit_round(torch.randn(shape, device="cuda", generator=g), fmt)


def _calls():
    x, w, b = _patterns((5, 37)), _patterns((11, 37), seed=2), _patterns((11,), seed=3)
    img, ker, kb = _patterns((2, 3, 10, 10)), _patterns((4, 3, 3, 3), seed=4), _patterns((4,), seed=5)
    dy = _patterns((2, 4, 5, 5), seed=6)
    d = pn.conv_desc((2, 3, 10, 10), (4, 3, 3, 3), (1, 1), (2, 2))
    f = torch.randn((3, 1, 7), device="cuda")
    idx = pn.posit_maxpool2d_fwd(img, "p8")[1]
    given = torch.zeros((5, 11), dtype=torch.int8, device="cuda")
    return {
        "gemm": lambda: pn.posit_gemm(x, w, "p8", "p16", trans_b=True, bias=b),
        "gemm given": lambda: pn.posit_gemm(x, w, "p8", "p8", trans_b=True, out=given),
        "gemm workspace": lambda: pn.posit_gemm(_patterns((300, 256)), _patterns((256, 300)), "p8", "p8"),
        "fwd": lambda: pn.posit_conv2d_fwd(img, ker, d, "p8", "p16", bias=kb),
        "bwd_data": lambda: pn.posit_conv2d_bwd_data(dy, ker, d, "p8", "p8"),
        "bwd_weight": lambda: pn.posit_conv2d_bwd_weight(dy, img, d, "p8", "p16", with_bias=True),
        "bwd_weight alone": lambda: pn.posit_conv2d_bwd_weight(dy, img, d, "p8", "p16"),
        "round": lambda: (pn.posit_round(f, "p12_2"), pn.posit_round(f.double(), "p32")),
        "convert": lambda: (pn.posit_convert(x, "p8", "f32"), pn.posit_convert(x, "p8", "p10_1")),
        "relu": lambda: (pn.posit_relu(x, "p8"), pn.posit_relu(x.view(torch.int8), "p8")),
        "relu_bwd": lambda: pn.posit_relu_bwd(x, _patterns((5, 37), "p16"), "p8", "p16"),
        "maxpool": lambda: pn.posit_maxpool2d_fwd(img, "p8", 5, 2) + (pn.posit_maxpool2d_bwd(_patterns(tuple(idx.shape)), idx, "p8"),),
        "avgpool": lambda: (pn.posit_avgpool2d_fwd(img, "p8", "p16"), pn.posit_avgpool2d_bwd(img, "p8", "p8", 2, 2)),
        "empty": lambda: (pn.posit_relu(x[:0], "p8"), pn.posit_gemm(x[:0], w, "p8", "p8", trans_b=True)),
        # refused, by whichever side
        "inner sizes": lambda: pn.posit_gemm(x, w, "p8", "p8"),
        "three dimensions": lambda: pn.posit_gemm(f, w, "p8", "p8"),
        "bias size": lambda: pn.posit_gemm(x, w, "p8", "p8", trans_b=True, bias=kb),
        "host tensor": lambda: pn.posit_gemm(x.cpu(), w, "p8", "p8", trans_b=True),
        "element size": lambda: pn.posit_relu(x, "p16"),
        "pitch": lambda: pn.posit_gemm(x[:, ::2], w[:, ::2], "p8", "p8", trans_b=True),
        "format": lambda: pn.posit_gemm(x, w, 57, "p8", trans_b=True),
        "format beyond 32 bits": lambda: pn.posit_gemm(x, w, 1 << 32, "p8", trans_b=True),
        "output format beyond 32 bits": lambda: pn.posit_gemm(x, w, "p8", 1 << 32, trans_b=True),
        "layer's format beyond 32 bits": lambda: pn.posit_conv2d_fwd(img, ker, d, "p8", 1 << 32, bias=kb),
        "format name": lambda: pn.posit_relu(x, "p9"),
        "source type": lambda: pn.posit_round(x, "p8"),
        "pool of a vector": lambda: pn.posit_maxpool2d_fwd(b, "p8"),
        "sizes": lambda: pn.posit_relu_bwd(x, w, "p8", "p8"),
        "no tensor": lambda: pn.posit_relu(None, "p8"),
    }


def _outcome(call):
    try:
        r = call()
    except Exception as e:
        return type(e), str(e)
    return [(t.dtype, tuple(t.shape), t.cpu().view(torch.uint8).tolist() if t.numel() else []) for t in (r if isinstance(r, tuple) else (r,))]


class _Recorder:
    """The native module, noting for each call which function was asked and whether it took the call."""

    def __init__(self, module):
        self.module, self.asked = module, []

    def __getattr__(self, name):
        def function(*args):
            r = getattr(self.module, name)(*args)
            self.asked.append((name, r is not None))
            return r
        return function


# the native functions that answer each call that succeeds (rounding makes some of the operands)
TAKEN = {"gemm": "gemm", "gemm given": "gemm", "gemm workspace": "round round gemm", "fwd": "conv", "bwd_data": "conv", "bwd_weight": "conv",
         "bwd_weight alone": "conv", "round": "round round", "convert": "convert convert", "relu": "relu relu", "relu_bwd": "round relu_bwd",
         "maxpool": "maxpool_fwd round maxpool_bwd", "avgpool": "avgpool avgpool", "empty": "relu gemm"}


def test_native_calls_do_what_the_python_code_does(monkeypatch):
    binding.load()
    calls = _calls()
    for name, call in calls.items():
        recorder = _Recorder(binding._native)
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", recorder)
            native = _outcome(call)
        with monkeypatch.context() as m:
            m.setattr(binding, "_native", None)
            assert native == _outcome(call), name
        assert isinstance(native, list) == (name in TAKEN), name
        if name in TAKEN:
            assert recorder.asked == [(f, True) for f in TAKEN[name].split()], name
        else:
            assert all(not taken for _, taken in recorder.asked), name  # nothing, or left to the Python code


def _longest_wait(call):
    """Seconds that another Python thread stood still at most while call ran, the median of nine."""
    waits = []
    for _ in range(9):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        started, stop, longest = threading.Event(), threading.Event(), [0.0]

        def run():
            last = time.perf_counter()
            started.set()
            while not stop.is_set():
                now = time.perf_counter()
                longest[0] = max(longest[0], now - last)
                last = now

        thread = threading.Thread(target=run)
        thread.start()
        started.wait()
        time.sleep(0.02)
        longest[0] = 0.0
        call()
        stop.set()
        thread.join()
        waits.append(longest[0])
    return sorted(waits)[4]


def test_other_threads_run_while_an_output_is_allocated(monkeypatch):
    """8 GiB fresh from the driver take about half a millisecond, in which the interpreter's lock is free as it is for torch.empty."""
    x = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
    convert = lambda: pn.posit_convert(x, "p8", "f64")
    convert()
    native = _longest_wait(convert)
    monkeypatch.setattr(binding, "_native", None)
    python = _longest_wait(convert)
    assert native < 2 * python + 1e-4, (native, python)


def test_native_calls_from_a_second_thread_on_its_own_stream():
    """Each thread works on its own current stream; outputs and workspaces belong to it."""
    a, b = _patterns((300, 256)), _patterns((256, 300), seed=2)
    want = pn.posit_relu(pn.posit_gemm(a, b, "p8", "p8"), "p8")
    torch.cuda.synchronize()
    got = [[], []]

    def run(out):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            assert binding._ready() == stream.cuda_stream
            for _ in range(50):
                out.append(pn.posit_relu(pn.posit_gemm(a, b, "p8", "p8"), "p8"))
        stream.synchronize()

    threads = [threading.Thread(target=run, args=(out,)) for out in got]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for out in got:
        assert len(out) == 50 and all(torch.equal(t, want) for t in out)
