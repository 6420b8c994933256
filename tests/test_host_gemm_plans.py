"""Which matrix products are accepted with which workspace, without a GPU: a call that passes the checks fails at its first
launch, one that does not is refused before it."""
import ctypes

import pytest
import torch

from paper_2105_00053_amd import binding

from test_host_logic import CODE, hc  # noqa: F401

EWORKSPACE, EHIP = 3, 4
no_gpu = pytest.mark.skipif(torch.cuda.is_available(), reason="the accepted calls would be launched on addresses that do not exist")
FAKE, NULL = ctypes.c_void_p(0x1000), ctypes.c_void_p(0)


def _gemm(fmt, M, N, K, bias, ws_bytes):
    c = CODE[fmt]
    return binding.load().posit_gemm(NULL, c, c, 0, 0, M, N, K, FAKE, K, FAKE, N, FAKE if bias else NULL, FAKE, N, FAKE if ws_bytes else NULL, ws_bytes)


@no_gpu
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


@no_gpu
@pytest.mark.parametrize("fmt", ["p8_1", "p8_2"])
def test_static_scratch_refuses_what_exceeds_it(fmt):
    assert binding.posit_gemm_workspace(fmt, fmt, 0, 0, 4096, 4096, 4096) > 72 << 20
    assert _static(fmt, 4096, 4096, 4096) == EWORKSPACE
    assert _static(fmt, 1024, 1024, 1024) == EHIP


@no_gpu
@pytest.mark.parametrize("fmt,M,N,K", [("p32", 4096, 4100, 1280), ("p32", 512, 512, 512), ("p16", 1024, 1024, 1024), ("p12_1", 1024, 1024, 1024)])
def test_static_scratch_takes_what_an_older_kernel_can_do(fmt, M, N, K):
    assert _static(fmt, M, N, K) == EHIP


@pytest.mark.parametrize("fmt", ["p8_1", "p8_2", "p10_1", "p12_1", "p16", "p32"])
def test_slices_of_a_reduction_and_where_their_sums_go(hc, fmt):  # noqa: F811
    """Every slice of either plane count has k blocks, the partial sums lie beside the planes and inside the workspace, and few
    tiles with a long reduction are cut for both counts (posit(8,1) and (8,2): for the narrow one only)."""
    out = (ctypes.c_int64 * 14)()
    hc.hostcheck_dig_plan.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 4 + [ctypes.c_void_p]
    for M, N, K in ((96, 96, 64), (96, 97, 4096), (100, 640, 1023), (115, 118, 10332), (97, 100, 16352), (787, 108, 4864), (300, 260, 1056), (512, 512, 512),
                    (1024, 1024, 1024), (1000, 1537, 500), (96, 700, 1040), (384, 400, 8192)):
        for limit in (-1, 72 << 20, 3 << 20):
            assert hc.hostcheck_dig_plan(CODE[fmt], M, N, K, limit, out)
            KB, s, kbps, off, per, planes, ws, wkbps, woff, wper, wplanes, room, rest, total = out[:]
            for slices, k, at, size, used in ((s, kbps, off, per, planes), (ws, wkbps, woff, wper, wplanes)):
                assert slices >= 1 and (slices - 1) * k < KB <= slices * k
                if slices > 1:
                    assert at % 16 == 0 and at >= used and at + slices * size <= total
                    assert at + slices * size <= room or at >= rest
            if fmt in ("p10_1", "p12_1", "p16"):
                tiles = ((M + 63) // 64) * ((N + 63) // 64)
                assert (s > 1) == (tiles <= 128 and KB >= 32)
                if limit < 0:
                    assert (ws > 1) == (s > 1)
                assert ws == 1 or limit < 0 or total <= max(limit, rest + s * per)


def test_which_products_take_32_by_32_tiles(hc):  # noqa: F811
    """posit(8,1), whose reduction is never cut: beyond one workgroup per compute unit only short reductions.  The other formats by
    their tiles, cut reductions aside."""
    hc.hostcheck_dig_small.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3
    for fmt, M, N, K, small in (("p8_1", 512, 512, 4096, 1), ("p8_1", 300, 800, 8192, 1), ("p8_1", 640, 704, 500, 1), ("p8_1", 640, 704, 501, 0),
                                ("p8_1", 640, 640, 1024, 0), ("p8_1", 333, 777, 4096, 0), ("p8_1", 448, 1024, 320, 1), ("p8_1", 448, 1024, 321, 0), ("p8_1", 128, 3584, 2048, 0),
                                ("p8_2", 640, 640, 1024, 1), ("p8_2", 640, 640, 2048, 0), ("p8_2", 640, 768, 300, 0), ("p12_1", 448, 1024, 768, 1),
                                ("p12_1", 448, 1024, 1024, 0), ("p16", 513, 1024, 100, 0), ("p32", 512, 512, 512, 0)):
        assert hc.hostcheck_dig_small(CODE[fmt], M, N, K) == small, (fmt, M, N, K)


def test_benchmark_names_the_kernel_that_the_library_takes(hc):  # noqa: F811
    import bench
    hc.hostcheck_p8_product.argtypes = [ctypes.c_int64] * 3
    names = {2: "p8_f6_gemm_kernel", 1: "p8_mfma_gemm_kernel"}
    for size in (512, 645, 646, 1024, 1920, 1921, 2048, 4096, 7168, 7169, 8192):
        kernel = bench.gemm_kernel_of(size)
        assert (kernel and kernel[0]) == names.get(hc.hostcheck_p8_product(size, size, size)), size
