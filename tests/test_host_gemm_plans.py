"""Which matrix products are accepted with which workspace, without a GPU: a call that passes the checks fails at its first
launch, one that does not is refused before it."""
import ctypes

import pytest
import torch

from paper_2105_00053_amd import binding

from test_host_logic import CODE

EWORKSPACE, EHIP = 3, 4
pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="the accepted calls would be launched on addresses that do not exist")
FAKE, NULL = ctypes.c_void_p(0x1000), ctypes.c_void_p(0)


def _gemm(fmt, M, N, K, bias, ws_bytes):
    c = CODE[fmt]
    return binding.load().posit_gemm(NULL, c, c, 0, 0, M, N, K, FAKE, K, FAKE, N, FAKE if bias else NULL, FAKE, N, FAKE if ws_bytes else NULL, ws_bytes)


def test_posit32_with_bias_needs_no_workspace():
    """The kernel with the quire in LDS serves it; without bias the digit planes take what the query answers."""
    M, N, K = 512, 512, 512
    need = binding.posit_gemm_workspace("p32", "p32", 0, 0, M, N, K)
    assert need > 0
    assert _gemm("p32", M, N, K, True, 0) == EHIP
    assert _gemm("p32", M, N, K, False, 0) == EWORKSPACE
    assert _gemm("p32", M, N, K, False, need - 1) == EWORKSPACE
    assert _gemm("p32", M, N, K, False, need) == EHIP


def _static(fmt, M, N, K):
    c = CODE[fmt]
    return binding.load().posit_gemm_static(NULL, c, c, 0, 0, M, N, K, FAKE, K, FAKE, N, NULL, FAKE, N)


@pytest.mark.parametrize("fmt", ["p8_1", "p8_2"])
def test_static_scratch_refuses_what_exceeds_it(fmt):
    assert binding.posit_gemm_workspace(fmt, fmt, 0, 0, 4096, 4096, 4096) > 72 << 20
    assert _static(fmt, 4096, 4096, 4096) == EWORKSPACE
    assert _static(fmt, 1024, 1024, 1024) == EHIP


@pytest.mark.parametrize("fmt,M,N,K", [("p32", 4096, 4100, 1280), ("p32", 512, 512, 512), ("p16", 1024, 1024, 1024), ("p12_1", 1024, 1024, 1024)])
def test_static_scratch_takes_what_an_older_kernel_can_do(fmt, M, N, K):
    assert _static(fmt, M, N, K) == EHIP
