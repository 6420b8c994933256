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
