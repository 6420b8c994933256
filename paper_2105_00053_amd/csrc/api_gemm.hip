// posit_gemm: quire-exact matrix product (paper Sec. 3.3; the Linear layer's
// forward, backward-data and backward-weight passes of Sec. 3.1 are its
// transposition cases).
#include <mutex>

#include "api_common.h"
#include "conv_p8.h"
#include "gemm_p8_w4.h"
#include "gemm_p8_f6.h"
#include "gemm_p8_mfma.h"
#include "gemm_dig_mfma.h"
#include "conv_b8.h"
#include "direct_gemm.h"
#include "gemm_bucket_pre.h"
#include "gemm_p16_window.h"
#include "gemm_p32_lds.h"

namespace pnn {

template <class F> struct GemmTile { static constexpr int TM = 4, TN = 4; };
template <> struct GemmTile<P32> { static constexpr int TM = 2, TN = 2; };

// posit<8,0> problems with both output dimensions beyond one small tile take the dot2 kernel
inline bool use_p8_kernel(int64_t M, int64_t N) { return M > 64 && N > 64; }

// ... and of those, the ones with too few 128 x 128 tiles to fill the chip go to the 64 x 64 kernel whose four waves
// split the reduction (larger products decode and pack their operands once instead)
inline bool use_p8_w4(int64_t M, int64_t N, int64_t K) { return use_p8_kernel(M, N) && p8_w4_fits(M, N, K) && !p8_packed_gemm_fits(M, N, K); }

// posit(8,1) / posit(8,2): the byte-gather kernel with fp64 buckets
template <class F>
constexpr bool is_b8() { return F::N == 8 && F::ES != 0; }

// Formats whose operands the digit kernels hold (posit<32,2> in a window; beyond it the LDS kernel does the work).
template <class F>
constexpr bool is_dig() { return F::N == 32 || (F::ES != 0 && DigFormat<F>::COVER); }

// Products that go to the integer matrix cores as base-256 digit planes, where the workspace may have up to `limit` bytes
// (posit(8,1) and posit(8,2) do not give way to their older kernel: beyond the limit the call is refused).
// Timed against the kernels that served before, drawn products with and without bias: of 1400 of the 16-bit containers, 2^16 to
// 2^31 multiply-adds, one was slower (860 x 286 x 112 with a bias, 28.6 us there, 30.6 here); of about 500
// posit<32,2> without bias none; of 700 posit(8,1) with a bias, 2^25 to 2^34, 6 by 7 to 11 % (500 to 770 tiles, of which the
// older kernel held three per compute unit, this one two), the mean 1.3 times as fast.
template <class F>
inline bool dig_gemm_fits(int64_t M, int64_t N, int64_t K, size_t limit) {
    if constexpr (!is_dig<F>()) return false;
    else {
        if (K > DIG_MAXK || M > ((int64_t)1 << 20) || N > ((int64_t)1 << 20)) return false;
        if (F::N == 8) {
            if (M < 128 || N < 128 || K < 256 || K > 8192 || M * N * K < ((int64_t)1 << 25) || ((M + 63) / 64) * ((N + 63) / 64) < 32) return false;
        } else if (F::N == 32) {
            if (!p32_lds_fits(M, N, K) || K < 256) return false;
        } else if (M < 96 || N < 96 || K < 64) {
            return false;
        }
        return F::N == 8 || dig_plan<F>(M, N, K, limit).total <= limit;
    }
}

// us of a product on the kernel that takes it if the direct one does not, where that is a matrix-core kernel or, for (10,2) and
// (12,2), the one with operands decoded once; fitted to products of 2^13 to 2^30 multiply-adds, off by 7 to 15 % (posit<8,0>: rows of
// odd lengths are decoded byte by byte, 208 x 813 x 1840 18.1 us there and 15.9 from the patterns).  Negative: another kernel.
// From 2^29 on the matrix-core kernels with digits written once are the faster ones throughout: zero.
template <class F>
inline double prepared_us(int64_t M, int64_t N, int64_t K, size_t limit) {
    const double g = (double)M * (double)N * (double)K / (1 << 30), k = 1e-3 * (double)K;
    if (F::N == 8 && F::ES == 0) return p8_f6_fits(M, N, K, limit) ? 0 : !p8_mfma_fits(M, N, K) ? -1 : g >= 0.5 ? 0 : p8_mfma_small(M, N) ? 11 + 5 * g + 1.2 * k + ((N | K) & 3 ? 5 : 0) : 17 + 19 * g;
    if (dig_gemm_fits<F>(M, N, K, limit)) {
        if (g >= 0.5) return 0;
        if (F::N == 8) return F::ES == 1 ? 16 + 15.7 * g + 3.8 * k : 17.5 + 20 * g + 2.4 * k;
        return 16.3 + 20 * g + 4 * k + 2.7 * (double)M * (double)N / (1 << 20);
    }
    if (bucket_pre_fits<F>(M, N, K)) return F::N == 10 ? 32 + 353 * g + 8 * k : 38 + 500 * g + 9 * k;
    return -1;
}

// Products that go to the matrix cores straight from their patterns, in one launch.  Against the kernels that serve otherwise, 500
// products of 8 to 4096 a side per format: faster by 1.6 (8 bits) and 4.6 to 6.3 times (10 to 16 bits) in the geometric mean, p16 48 x 368 x 340
// 161 -> 8.4 us, posit<8,0> 850 x 160 x 1632 78 -> 9.7; what stays behind: estimates within a tenth of each other (8 bits with short table
// entries: a fifth, strided operands cost them more), products of few outputs of the 8-bit formats (a thread group per output: 12 x 11 x 3737 7.8 us
// there, 9.7 here) and reductions too short for a k block of 64 (1279 x 2486 x 11, p16, 52 and 57).
template <class F>
inline DirectPlan direct_gemm_plan(int64_t M, int64_t N, int64_t K, size_t limit) {
    const DirectPlan none{DIRECT_NONE, 1, 0, 0};
    if constexpr (F::N > 16) return none;
    else {
        if (K < 16 && M * N > ((int64_t)1 << 19)) return none;
        if (F::N == 8) {
            if (M * N < 2048 || (M * N < 4096 && K > 1024)) return none;
            if (K < 32 && M * N <= ((int64_t)1 << 19) && (F::ES == 2 || N < 32)) return none;
        }
        double us;
        const DirectPlan p = direct_plan<F>(M, N, K, &us);
        if (p.variant == DIRECT_NONE || p.ws_bytes > limit) return none;
        const double prepared = prepared_us<F>(M, N, K, limit);
        // other kernels: the vector ALU at some 10 TMAC/s and less
        if (prepared < 0) return K <= 4096 || (double)M * (double)N * (double)K < 1e9 ? p : none;
        return us < (F::N == 8 && F::ES < 2 ? 0.8 : 0.92) * prepared ? p : none;
    }
}

// posit<32,2> below the tiles from which the digit planes and the LDS kernel serve: in one launch on the matrix cores, the window of bits taken by each
// workgroup for itself.  Against the general kernel, us: 8 x 8 x 4 19.9 and 8.3, 64 x 64 x 256 215 and 9.6, 432 x 432 x 2048 803 and 95; operands
// that span more than the window, 64 x 64 x 1024 220 and 90, x 2048 224 and 176, 16 x 16 x 4000 235 and 345 (N(0, 1): 55), hence the end of the
// reduction below 256 tiles; from there on the general kernel is full: 256 x 256 x 11904 1469 and 174 (1466 and 1070), 350 x 260 x 3000 579 and 92 (579
// and 565).  432 x 432 x 16, three rounds of workgroups, 20.5 and 23.  Where the other two serve they are faster: 500 x 500 x 500 35 and 45.
inline bool p32_direct_fits(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((M + 15) / 16) * ((N + 15) / 16);
    return K >= 1 && K <= (tiles < 256 ? 2048 : DIRECT_MAXK) && M <= 16384 && N <= 16384 && tiles < (K < 32 ? 512 : 768);
}

// Cut of the kernels that serve where the direct one does not.
template <class F>
GemmPlan prepared_plan(int64_t M, int64_t N, int64_t K, size_t limit = SIZE_MAX) {
    if (dig_gemm_fits<F>(M, N, K, limit)) {
        GemmPlan p;
        p.splits = 1; p.k_per_split = K; p.ws_bytes = 0;
        if constexpr (is_dig<F>()) p.ws_bytes = dig_plan<F>(M, N, K, limit).total;
        return p;
    }
    if constexpr (is_b8<F>()) {
        if (p8_small_gemm_fits(M, N, K)) {  // one thread group per output: no workspace
            GemmPlan p;
            p.splits = 1; p.k_per_split = K; p.ws_bytes = 0;
            return p;
        }
        if (M < ((int64_t)1 << 31) && N < ((int64_t)1 << 31) && K < ((int64_t)1 << 31)) return b8_conv_plan<F>((int)M, (int)N, (int)K);
    }
    if ((F::N == 8 && F::ES == 0) && p8_small_gemm_fits(M, N, K)) {  // one thread group per output: no workspace
        GemmPlan p;
        p.splits = 1; p.k_per_split = K; p.ws_bytes = 0;
        return p;
    }
    if ((F::N == 8 && F::ES == 0) && p8_f6_fits(M, N, K, limit)) {  // digits for the 6-bit floating-point matrix cores, or planes as below
        GemmPlan p;
        p.splits = 1; p.k_per_split = K; p.ws_bytes = p8_f6_layout(M, N, K).total();
        return p;
    }
    if ((F::N == 8 && F::ES == 0) && p8_mfma_fits(M, N, K)) {  // digit planes of both operands for the integer matrix cores
        GemmPlan p;
        p.splits = 1; p.k_per_split = K; p.ws_bytes = p8_mfma_layout(M, N, K).total();
        return p;
    }
    if ((F::N == 8 && F::ES == 0) && use_p8_w4(M, N, K)) return p8_w4_plan(M, N, K).gemm;  // the reduction is cut inside the workgroup first
    if ((F::N == 8 && F::ES == 0) && use_p8_kernel(M, N)) {
        GemmPlan p = plan_split(M, N, K, P8_BM, P8_BN, 1, P8_KT);
        if (p8_packed_gemm_fits(M, N, K)) p.ws_bytes += p8_packed_layout(M, N, K).total();  // operands packed once, ahead of the split partials
        return p;
    }
    // other posit<8,0> shapes go to the gather kernel (tile chosen per shape); the plan does not depend on pitches
    if ((F::N == 8 && F::ES == 0) && M < ((int64_t)1 << 31) && N < ((int64_t)1 << 31) && K < ((int64_t)1 << 31)) return p8_conv_plan((int)M, (int)N, (int)K);
    if (F::N == 32 && p32_lds_fits(M, N, K)) {  // the quire of every output lives in LDS for the whole reduction: no workspace
        GemmPlan p;
        p.splits = 1; p.k_per_split = K; p.ws_bytes = 0;
        return p;
    }
    if (F::N == 16 && pw_fits(M, N, K)) return pw_plan(M, N, K).gemm;          // posit<16,1>: operands decoded once, two buckets + outlier bitmaps
    if (bucket_pre_fits<F>(M, N, K)) return bucket_pre_plan<F>(M, N, K).gemm;  // operands decoded once into the workspace
    return plan_split(M, N, K, 16 * GemmTile<F>::TM, 16 * GemmTile<F>::TN, Arith<F>::L);
}

// What a call asks for: the query does not know the pitches, and operands beyond the direct kernel's offsets go to the others.
template <class F>
size_t gemm_workspace(int64_t M, int64_t N, int64_t K, size_t limit = SIZE_MAX) {
    const size_t a = prepared_plan<F>(M, N, K, limit).ws_bytes, b = direct_gemm_plan<F>(M, N, K, limit).ws_bytes;
    return a > b ? a : b;
}

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
