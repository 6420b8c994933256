// Which kernel takes a matrix product and what workspace it asks for: api_gemm.hip dispatches by it.
#pragma once

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
// (12,2), the one with operands decoded once; fitted to products of 2^13 to 2^30 multiply-adds, off by 7 to 15 %.  posit<8,0>: 207 products of 2^25 to
// 2^29, off by 14 % with 32 x 32 tiles, 10 % with 64 x 64, whose fewer outputs bring longer reductions and slices (811 x 1936 x 256 14.2 us, 6768 x 256 x 272 15.7).
// Negative: another kernel.  From 2^29 on the matrix-core kernels with digits written once are the faster ones throughout: zero.
template <class F>
inline double prepared_us(int64_t M, int64_t N, int64_t K, size_t limit) {
    const double g = (double)M * (double)N * (double)K / (1 << 30), k = 1e-3 * (double)K, mn = (double)M * (double)N / (1 << 20);
    if (F::N == 8 && F::ES == 0) {
        if (p8_f6_fits(M, N, K, limit)) return 0;
        if (!p8_mfma_fits(M, N, K)) return -1;
        return g >= 0.5 ? 0 : p8_mfma_small(M, N, K) ? 7 + 11 * g + 1.2 * k + 1.9 * mn : 15 + 17 * g + 0.2 * k - 5 * mn;
    }
    if (dig_gemm_fits<F>(M, N, K, limit)) {
        if (g >= 0.5) return 0;
        if (F::N == 8) return F::ES == 1 ? 16 + 15.7 * g + 3.8 * k : 17.5 + 20 * g + 2.4 * k;
        return 16.3 + 20 * g + 4 * k + 2.7 * mn;
    }
    if (bucket_pre_fits<F>(M, N, K)) return F::N == 10 ? 32 + 353 * g + 8 * k : 38 + 500 * g + 9 * k;
    return -1;
}

// Most outputs of a reduction of up to half a k block: the block's other half is zeros here, the general kernel stops at a multiple of 16.  us, general
// kernel and this one, N(0, 1): 2048 x 2048 x 16, posit<16,1>, 51.4 and 74.9, (12,1) 43.8 and 64.1, (12,2) 94 and 132, (10,2) 51 and 70, (10,1)
// 42.7 and 40.3 (the second operand transposed 1.25 times as long); x 31 (12,1) 57.0 and 57.8, (12,2) 126 and 129, posit<16,1> 70.9 and 68.8, at 4096 x 4096 201 and 220,
// 498 and 506, 254 and 261, (10,2) 256 and 248, (10,1) 197 and 127; x 33 all faster here (posit<16,1> 1024 x 1024 0.61 of the time, 3000 x 3000 0.76).
template <class F>
constexpr int64_t direct_short_outputs(int64_t K) {
    if (K > 32 || (F::N == 8 && K >= 16)) return INT64_MAX;
    if (K <= 16 || (F::N == 12 && F::ES == 2)) return (int64_t)1 << 19;
    return F::N == 10 ? INT64_MAX : (int64_t)1 << 21;
}

// posit<8,0> below the reductions of the matrix-core kernels (256): from 3 x 2^20 outputs on the vector ALU's 128 x 128 tiles have a full round of workgroups, and
// the kernel straight from the patterns, bound by its conversions and stores, has no latency left to save.  us, those tiles and direct: 32 indices,
// 1448 x 1448 123 and 18 (16 indices 34 and 15), 2048 x 2048 14 and 27, 4096 x 4096 27 and 82, 8192 x 8192 80 and 318; 64, 3191 x 2865 35 and 44, 4096 x 4096 36 and 76; 129,
// 2048 x 2048 24 and 30, 4096 x 4096 75 and 118; 255, 1500 x 1500 41 and 21, 4096 x 4096 112 and 136.  1190 products of 2^18 to 2^26.5 outputs, three orders:
// 486 of them go direct, 8 of these are more than 3 % behind (at most 6); without a limit 485 were, by up to 4 times.  Sides of at most 64 do not have those tiles.
inline bool p8_direct_outputs(int64_t M, int64_t N, int64_t K) { return !use_p8_kernel(M, N) || K >= 256 || M * N <= ((int64_t)3 << 20); }

// Products that go to the matrix cores straight from their patterns, in one launch.  Against the kernels that serve otherwise, 500
// products of 8 to 4096 a side per format: faster by 1.6 (8 bits) and 4.6 to 6.3 times (10 to 16 bits) in the geometric mean, p16 48 x 368 x 340
// 161 -> 8.4 us, posit<8,0> 850 x 160 x 1632 78 -> 9.7; what stays behind: estimates close to each other (direct_pays), products of few outputs of the 8-bit formats (a thread group per output: 12 x 11 x 3737 7.8 us
// there, 9.7 here) and reductions too short for a k block of 64: direct_short_outputs, and of few products of 8 bits, for which a workgroup's table and the barriers around it are
// the call (posit<8,0>, us in a replayed graph, where launches do not hide it, others and direct: 48 x 48 x 4 2.4 and 3.8, 250 x 250 x 16 3.4 and 4.4, 700 x 700 x 8 4.7 and 5.1, x 12 5.9 and
// 5.2; (8,1) 128 x 128 x 8 3.1 and 4.4; 250 x 250 x 32 6.1 and 4.6; posit<8,0> 2823 x 6 x 32 4.2 and 5.5, 4194 x 5 x 40 4.6 and 5.6).
template <class F>
inline DirectPlan direct_gemm_plan(int64_t M, int64_t N, int64_t K, size_t limit) {
    const DirectPlan none{DIRECT_NONE, 1, 0, 0};
    if constexpr (F::N > 16) return none;
    else {
        if (M * N > direct_short_outputs<F>(K)) return none;
        if (F::N == 8) {
            if (M * N < 2048 || (M * N < 4096 && K > 1024)) return none;
            if (K < 32 && M * N <= ((int64_t)1 << 19) && (F::ES == 2 || N < 32)) return none;
            if ((K < 30 && M * N * K < 5000000) || (N <= 16 && K < 48)) return none;
            if (F::ES == 0 && !p8_direct_outputs(M, N, K)) return none;
        }
        double us;
        const DirectPlan p = direct_plan<F>(M, N, K, &us);
        if (p.variant == DIRECT_NONE || p.ws_bytes > limit) return none;
        const double prepared = prepared_us<F>(M, N, K, limit);
        // other kernels: the vector ALU at some 10 TMAC/s and less, thin posit<8,0> products and those of few outputs among them
        if (prepared < 0) return K <= 4096 || (double)M * (double)N * (double)K < 1e9 ? p : none;
        return direct_pays(us, (double)M * (double)N * (double)K, prepared) ? p : none;
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

}  // namespace pnn
