// posit_gemm: quire-exact matrix product (paper Sec. 3.3; the Linear layer's
// forward, backward-data and backward-weight passes of Sec. 3.1 are its
// transposition cases).
#include <mutex>

#include "gemm_choice.h"

namespace pnn {

template <class F>
int gemm_dispatch(hipStream_t st, int fout, int transA, int transB, int64_t M, int64_t N, int64_t K,
                  const void* A, int64_t lda, const void* B, int64_t ldb, const void* bias, void* C, int64_t ldc,
                  void* ws, size_t ws_bytes, size_t limit) {
    typedef typename Storage<F::N>::T T;
    constexpr int TM = GemmTile<F>::TM, TN = GemmTile<F>::TN;
    const GemmPlan plan = prepared_plan<F>(M, N, K, limit);
    // posit<32,2> with a bias: the LDS kernel, whose quire takes it at any scale and which needs no workspace
    const bool use_dig = dig_gemm_fits<F>(M, N, K, limit) && (F::N != 32 || !bias);
    const bool no_ws = F::N == 32 && bias && p32_lds_fits(M, N, K);
    if (plan.ws_bytes > 0 && !no_ws && (!ws || ws_bytes < plan.ws_bytes)) return PNN_EWORKSPACE;
    RowMajorOut out;
    out.ld = ldc;
    hipError_t e;
    if constexpr (F::N <= 16) {
        const DirectPlan direct = direct_gemm_plan<F>(M, N, K, limit);
        if (direct.variant != DIRECT_NONE && (direct.ws_bytes == 0 || (ws && ws_bytes >= direct.ws_bytes)) && direct_extent_fits(transA, transB, M, N, K, lda, ldb, sizeof(T)))
            return hip_status(launch_direct_gemm<F>(st, direct, transA, transB, M, N, K, A, lda, B, ldb, bias, C, ldc, fout, ws));
    }
    if constexpr (F::N == 32) {
        if (p32_direct_fits(M, N, K) && !bias && direct_extent_fits(transA, transB, M, N, K, lda, ldb, sizeof(T)))
            return hip_status(launch_direct_p32(st, transA, transB, M, N, K, A, lda, B, ldb, C, ldc, fout));
    }
    const int* served = nullptr;  // on the device: non-zero when the digit kernels did the work
    if constexpr (is_dig<F>()) {
        if (use_dig) {
            const DigInfo* decision;
            e = launch_dig_gemm<F>(st, transA, transB, A, lda, B, ldb, bias, C, ldc, fout, M, N, K, ws, limit, &decision);
            if (e != hipSuccess || DigFormat<F>::COVER) return hip_status(e);
            served = &decision->np;
        }
    }
    if ((F::N == 8 && F::ES == 0) && p8_small_gemm_fits(M, N, K))
        return hip_status(launch_p8_small_gemm(st, transA, transB, (const uint8_t*)A, lda, (const uint8_t*)B, ldb, (const uint8_t*)bias, C, ldc,
                                               fout, M, N, K));
    if ((F::N == 8 && F::ES == 0) && p8_f6_fits(M, N, K, limit))
        return hip_status(launch_p8_f6_gemm(st, transA, transB, (const uint8_t*)A, lda, (const uint8_t*)B, ldb, (const uint8_t*)bias, C, ldc, fout, M, N,
                                            K, ws));
    if ((F::N == 8 && F::ES == 0) && p8_mfma_fits(M, N, K))
        return hip_status(launch_p8_mfma_gemm(st, transA, transB, (const uint8_t*)A, lda, (const uint8_t*)B, ldb, (const uint8_t*)bias, C, ldc, fout,
                                              M, N, K, ws));
    if ((F::N == 8 && F::ES == 0) && use_p8_w4(M, N, K)) {
        const uint8_t* a8 = (const uint8_t*)A;
        const uint8_t* b8 = (const uint8_t*)B;
        const uint8_t* bias8 = (const uint8_t*)bias;
        if (!transA && !transB) e = launch_p8_gemm_w4<true, false>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws);
        else if (!transA && transB) e = launch_p8_gemm_w4<true, true>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws);
        else if (transA && !transB) e = launch_p8_gemm_w4<false, false>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws);
        else e = launch_p8_gemm_w4<false, true>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws);
        return hip_status(e);
    }
    if ((F::N == 8 && F::ES == 0) && use_p8_kernel(M, N) && p8_packed_gemm_fits(M, N, K)) {
        return hip_status(launch_p8_gemm_packed(st, transA, transB, (const uint8_t*)A, lda, (const uint8_t*)B, ldb, (const uint8_t*)bias, C, ldc,
                                                fout, M, N, K, ws, plan));
    }
    if ((F::N == 8 && F::ES == 0) && use_p8_kernel(M, N)) {
        const uint8_t* a8 = (const uint8_t*)A;
        const uint8_t* b8 = (const uint8_t*)B;
        const uint8_t* bias8 = (const uint8_t*)bias;
        // operand tiles are (rows x k): A's rows are m, B's rows are n; B is k-contiguous only when transposed
        if (!transA && !transB) e = launch_p8_gemm<true, false>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws, plan);
        else if (!transA && transB) e = launch_p8_gemm<true, true>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws, plan);
        else if (transA && !transB) e = launch_p8_gemm<false, false>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws, plan);
        else e = launch_p8_gemm<false, true>(st, a8, lda, b8, ldb, bias8, C, ldc, fout, M, N, K, ws, plan);
        return hip_status(e);
    }
    if ((F::N == 8 && F::ES == 0) && p8_gemm_as_gather_fits(transA, transB, M, N, K, lda, ldb)) {
        const P8ConvProblem p = p8_gemm_problem(transA, transB, (int)M, (int)N, (int)K, A, (int)lda, B, (int)ldb, ldc);
        return hip_status(p8_conv_launch_rowmajor(st, p, (const uint8_t*)bias, C, fout, ws, plan, ldc));
    }
    if constexpr (is_b8<F>()) {
        if (p8_small_gemm_fits(M, N, K))
            return hip_status(launch_b8_small_gemm<F>(st, transA, transB, (const uint8_t*)A, lda, (const uint8_t*)B, ldb, (const uint8_t*)bias, C,
                                                      ldc, fout, M, N, K));
        if (p8_gemm_as_gather_fits(transA, transB, M, N, K, lda, ldb)) {
            const P8ConvProblem p = p8_gemm_problem(transA, transB, (int)M, (int)N, (int)K, A, (int)lda, B, (int)ldb, ldc);
            RowMajorOut mo{ldc};
            return hip_status(b8_conv_launch<F>(st, p, (const uint8_t*)bias, C, fout, ws, plan, mo));
        }
    }
    if constexpr (F::N == 32) {
        if (p32_lds_fits(M, N, K)) {
            if (!transA && !transB) {
                MatrixOperand<T, true> a{(const T*)A, lda, M, K};
                MatrixOperand<T, false> b{(const T*)B, ldb, N, K};
                return hip_status(launch_p32_lds_gemm(st, a, b, M, N, K, bias, C, ldc, fout, served));
            } else if (!transA && transB) {
                MatrixOperand<T, true> a{(const T*)A, lda, M, K};
                MatrixOperand<T, true> b{(const T*)B, ldb, N, K};
                return hip_status(launch_p32_lds_gemm(st, a, b, M, N, K, bias, C, ldc, fout, served));
            } else if (transA && !transB) {
                MatrixOperand<T, false> a{(const T*)A, lda, M, K};
                MatrixOperand<T, false> b{(const T*)B, ldb, N, K};
                return hip_status(launch_p32_lds_gemm(st, a, b, M, N, K, bias, C, ldc, fout, served));
            } else {
                MatrixOperand<T, false> a{(const T*)A, lda, M, K};
                MatrixOperand<T, true> b{(const T*)B, ldb, N, K};
                return hip_status(launch_p32_lds_gemm(st, a, b, M, N, K, bias, C, ldc, fout, served));
            }
        }
    }
    if constexpr (F::N == 16) {
        if (pw_fits(M, N, K)) return hip_status(launch_pw_gemm(st, transA, transB, A, lda, B, ldb, bias, C, ldc, fout, M, N, K, ws));
    }
    if constexpr (bucket_pre_format<F>()) {
        if (bucket_pre_fits<F>(M, N, K))
            return hip_status(launch_bucket_pre_gemm<F>(st, transA, transB, A, lda, B, ldb, bias, C, ldc, fout, M, N, K, ws));
    }
    // op(A)[i,k]: k contiguous unless transA.  op(B)[k,j] seen as rows j: k contiguous only when transB.
    if (!transA && !transB) {
        MatrixOperand<T, true> a{(const T*)A, lda, M, K};
        MatrixOperand<T, false> b{(const T*)B, ldb, N, K};
        e = launch_quire_gemm<F, decltype(a), decltype(b), RowMajorOut, TM, TN>(st, a, b, out, M, N, K, bias, C, fout, ws, plan);
    } else if (!transA && transB) {
        MatrixOperand<T, true> a{(const T*)A, lda, M, K};
        MatrixOperand<T, true> b{(const T*)B, ldb, N, K};
        e = launch_quire_gemm<F, decltype(a), decltype(b), RowMajorOut, TM, TN>(st, a, b, out, M, N, K, bias, C, fout, ws, plan);
    } else if (transA && !transB) {
        MatrixOperand<T, false> a{(const T*)A, lda, M, K};
        MatrixOperand<T, false> b{(const T*)B, ldb, N, K};
        e = launch_quire_gemm<F, decltype(a), decltype(b), RowMajorOut, TM, TN>(st, a, b, out, M, N, K, bias, C, fout, ws, plan);
    } else {
        MatrixOperand<T, false> a{(const T*)A, lda, M, K};
        MatrixOperand<T, true> b{(const T*)B, ldb, N, K};
        e = launch_quire_gemm<F, decltype(a), decltype(b), RowMajorOut, TM, TN>(st, a, b, out, M, N, K, bias, C, fout, ws, plan);
    }
    return hip_status(e);
}

}  // namespace pnn

using namespace pnn;

extern "C" size_t posit_gemm_workspace(int fin, int fout, int transA, int transB, int64_t M, int64_t N, int64_t K) {
    (void)fout; (void)transA; (void)transB;
    if (!is_posit(fin) || M <= 0 || N <= 0 || K < 0) return 0;
    PNN_DISPATCH_POSIT(fin, return gemm_workspace<F>(M, N, K))
    return 0;
}

// Argument checks shared by the entry points below.  *launch is set when there is work to do.
static int gemm_check_args(int fin, int fout, int transA, int transB, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                           const void* B, int64_t ldb, const void* C, int64_t ldc, bool* launch) {
    *launch = false;
    if (!is_posit(fin) || !is_posit(fout) || M < 0 || N < 0 || K < 0) return PNN_EINVAL;
    if (M == 0 || N == 0) return PNN_OK;
    if (!C || ldc < N) return PNN_EINVAL;
    if (K > 0) {
        if (!A || !B) return PNN_EINVAL;
        if (lda < (transA ? M : K) || ldb < (transB ? K : N)) return PNN_EINVAL;
    }
    if (M >= ((int64_t)1 << 31) || N >= ((int64_t)1 << 31) || K >= ((int64_t)1 << 31) || M * N >= ((int64_t)1 << 40)) return PNN_EUNSUPPORTED;
    *launch = true;
    return PNN_OK;
}

extern "C" int posit_gemm(void* stream, int fin, int fout, int transA, int transB, int64_t M, int64_t N, int64_t K,
                          const void* A, int64_t lda, const void* B, int64_t ldb, const void* bias, void* C, int64_t ldc,
                          void* workspace, size_t workspace_bytes) {
    bool launch;
    const int rc = gemm_check_args(fin, fout, transA, transB, M, N, K, A, lda, B, ldb, C, ldc, &launch);
    if (!launch) return rc;
    if (workspace && ((uintptr_t)workspace & 15u) != 0) return PNN_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    discard_stale_hip_error();
    PNN_DISPATCH_POSIT(fin, return gemm_dispatch<F>(st, fout, transA, transB, M, N, K, A, lda, B, ldb, bias, C, ldc, workspace, workspace_bytes, SIZE_MAX))
    return PNN_EINVAL;
}

// ---- posit_gemm for callers that cannot allocate device memory ----
//
// The workspace of posit_gemm (partial quires of a split reduction, packed operands) lives in a
// fixed array inside the library's code object instead of a caller's buffer.  Each GPU the library
// runs on holds its own copy of the array at its own address; in host code the array's name is
// only a handle for hipGetSymbolAddress, never a device address, so the address is looked up once
// per device (first call with that device current) and that pointer is what the kernels receive.

static __device__ __align__(256) unsigned char scratch[PNN_GEMM_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
void* g_scratch_ptr[MAX_DEVICES];  // per device: device address of `scratch`, null until looked up
std::mutex g_scratch_mutex;

// Device address of the current device's copy of `scratch`.
int scratch_address(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return PNN_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PNN_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PNN_OK;
}
}  // namespace

extern "C" int posit_gemm_static(void* stream, int fin, int fout, int transA, int transB, int64_t M, int64_t N, int64_t K,
                                 const void* A, int64_t lda, const void* B, int64_t ldb, const void* bias, void* C, int64_t ldc) {
    bool launch;
    const int rc = gemm_check_args(fin, fout, transA, transB, M, N, K, A, lda, B, ldb, C, ldc, &launch);
    if (!launch) return rc;
    // digit planes that want more than the fixed array give way to an older kernel that does not (see dig_gemm_fits)
    const size_t limit = PNN_GEMM_STATIC_SCRATCH_BYTES;
    size_t need = 0;
    PNN_DISPATCH_POSIT(fin, need = gemm_workspace<F>(M, N, K, limit))
    if (need > PNN_GEMM_STATIC_SCRATCH_BYTES) return PNN_EWORKSPACE;  // beyond the fixed array: posit_gemm with a caller's workspace
    void* ws = nullptr;
    if (need > 0) {
        const int rs = scratch_address(&ws);
        if (rs != PNN_OK) return rs;
    }
    hipStream_t st = (hipStream_t)stream;
    discard_stale_hip_error();
    const size_t ws_bytes = need > 0 ? (size_t)PNN_GEMM_STATIC_SCRATCH_BYTES : 0;
    PNN_DISPATCH_POSIT(fin, return gemm_dispatch<F>(st, fout, transA, transB, M, N, K, A, lda, B, ldb, bias, C, ldc, ws, ws_bytes, limit))
    return PNN_EINVAL;
}
