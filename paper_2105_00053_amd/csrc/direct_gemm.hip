// Matrix products on direct_kernel (direct_mfma.h).
#include "direct_gemm.h"

#include "direct_mfma.h"

namespace pnn {

template <class F>
hipError_t launch_direct_gemm(hipStream_t st, const DirectPlan& p, int transA, int transB, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                              const void* B, int64_t ldb, const void* bias, void* C, int64_t ldc, int fout, void* workspace) {
    typedef typename Storage<F::N>::T T;
    constexpr uint32_t E = sizeof(T);
    const DirectMatrix<T> a{(const T*)A, transA ? E : (uint32_t)lda * E, transA ? (uint32_t)lda * E : E, (int)M};
    const DirectMatrix<T> b{(const T*)B, transB ? (uint32_t)ldb * E : E, transB ? E : (uint32_t)ldb * E, (int)N};
    return launch_direct<F>(st, p, a, b, RowMajorOut{ldc}, (int)M, (int)N, (int)K, bias, C, fout, workspace);
}

hipError_t launch_direct_p32(hipStream_t st, int transA, int transB, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                             void* C, int64_t ldc, int fout) {
    typedef DirectMatrix<uint32_t> Op;
    const Op a{(const uint32_t*)A, transA ? 4u : (uint32_t)lda * 4u, transA ? (uint32_t)lda * 4u : 4u, (int)M};
    const Op b{(const uint32_t*)B, transB ? (uint32_t)ldb * 4u : 4u, transB ? 4u : (uint32_t)ldb * 4u, (int)N};
    const int64_t tiles_m = (M + 15) / 16, tiles_n = (N + 15) / 16;
    hipLaunchKernelGGL(direct_p32_kernel<Op>, dim3((unsigned)(tiles_m * tiles_n)), dim3(512), 0, st, a, b, (int)M, (int)N, (int)K, C, ldc, fout, (int)tiles_n);
    return hipGetLastError();
}

#define PNN_DIRECT_GEMM(F)                                                                                                                        \
    template hipError_t launch_direct_gemm<F>(hipStream_t, const DirectPlan&, int, int, int64_t, int64_t, int64_t, const void*, int64_t, const void*, \
                                              int64_t, const void*, void*, int64_t, int, void*);
PNN_DIRECT_GEMM(P8)
PNN_DIRECT_GEMM(P8_1)
PNN_DIRECT_GEMM(P8_2)
PNN_DIRECT_GEMM(P10_1)
PNN_DIRECT_GEMM(P10_2)
PNN_DIRECT_GEMM(P12_1)
PNN_DIRECT_GEMM(P12_2)
PNN_DIRECT_GEMM(P16)

}  // namespace pnn
