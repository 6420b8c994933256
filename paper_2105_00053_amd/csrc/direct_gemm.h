// Which products take direct_kernel (direct_mfma.h) and how they are cut, and their launch.  The kernels are in a unit of
// their own (direct_gemm.hip).
#pragma once

#include "quire_gemm.h"

namespace pnn {

constexpr int DIRECT_MAXK = 11904;                  // longest reduction of one workgroup: 11 digit pairs * 2^14 * K < 2^31
constexpr int64_t DIRECT_EXTENT = (int64_t)1 << 31;  // most bytes of an operand: offsets are 32 bits

// Waves of a workgroup: 16 x 16 outputs and 8 or 4 waves that share the reduction; 64 x 16 and a wave for each block; 32 x 32 with
// every pattern converted once.
enum DirectVariant { DIRECT_NONE, DIRECT_W8, DIRECT_W4, DIRECT_COL, DIRECT_SHARED };

struct DirectPlan {
    int variant;
    int splits, k_per_split;
    size_t ws_bytes;
};

// us of a call: base + unit per 1000 (tile, k block of 64) + step per k block one wave goes through + group per 1000 workgroups.  Fitted to
// 500 products per format of 8 to 4096 a side (and, sliced, those of up to 2^16 outputs); off by 11 to 15 % (root mean square).
struct DirectCost { float base, unit, step, group; };
constexpr int DIRECT_SLICED = 4;  // fifth row: 16 x 16, eight waves, slices and the merging launch
template <class F>
inline const DirectCost* direct_cost() {
    static const DirectCost COST[8][5] = {
        {{5.61f, 0.335f, 0.447f, 2.93f}, {5.56f, 0.32f, 0.51f, 1.21f}, {5.4f, 1.01f, 0.735f, 2.79f}, {5.35f, 0.611f, 0.675f, 2.59f}, {8.88f, 0.273f, 0.f, 2.29f}},       // posit<8,0>
        {{5.32f, 0.352f, 0.693f, 4.01f}, {5.4f, 0.356f, 0.604f, 1.82f}, {5.47f, 1.1f, 0.842f, 3.84f}, {5.11f, 0.844f, 0.896f, 4.41f}, {8.85f, 0.421f, 0.f, 3.08f}},      // (8,1)
        {{4.76f, 0.455f, 1.22f, 5.17f}, {4.99f, 0.463f, 0.963f, 3.27f}, {5.69f, 1.3f, 1.15f, 6.21f}, {4.49f, 1.51f, 1.58f, 11.f}, {8.15f, 0.66f, 0.594f, 4.73f}},        // (8,2)
        {{4.85f, 0.491f, 1.15f, 4.89f}, {5.02f, 0.467f, 1.03f, 2.53f}, {5.72f, 1.29f, 1.23f, 5.19f}, {4.82f, 1.13f, 1.32f, 5.94f}, {8.71f, 0.609f, 0.503f, 4.12f}},      // (10,1)
        {{4.02f, 0.837f, 1.87f, 12.9f}, {4.33f, 0.738f, 1.68f, 6.89f}, {6.12f, 1.99f, 1.71f, 10.2f}, {5.98f, 3.14f, 1.69f, 18.9f}, {9.32f, 1.19f, 1.22f, 12.7f}},        // (10,2)
        {{4.68f, 0.543f, 1.32f, 5.87f}, {4.82f, 0.496f, 1.23f, 4.45f}, {6.17f, 1.56f, 1.13f, 8.94f}, {4.61f, 1.6f, 1.48f, 11.4f}, {8.58f, 0.752f, 0.556f, 4.92f}},       // (12,1)
        {{4.07f, 0.993f, 2.43f, 16.2f}, {4.92f, 1.3f, 1.69f, 17.4f}, {6.93f, 3.5f, 1.81f, 23.8f}, {6.76f, 3.58f, 1.94f, 22.2f}, {10.1f, 1.51f, 1.4f, 15.4f}},            // (12,2)
        {{2.56f, 1.56f, 3.7f, 12.2f}, {3.85f, 1.37f, 2.35f, 6.69f}, {5.51f, 4.17f, 2.45f, 9.68f}, {3.6f, 2.96f, 2.92f, 13.4f}, {6.93f, 2.43f, 2.64f, 8.45f}},            // posit<16,1>
    };
    return COST[F::N == 8 ? F::ES : F::N == 10 ? 2 + F::ES : F::N == 12 ? 4 + F::ES : 7];
}

template <class F>
constexpr int direct_shared_groups() { return 2 * F::MAXS + 1 > 62 ? 1 : 2; }  // of four waves; more than eight planes take the LDS of two groups

// Rows and columns of a workgroup, waves that share its reduction; waves.
struct DirectShape { int tr, tc, kg, waves; };
template <class F>
constexpr DirectShape direct_shape(int variant) {
    return variant == DIRECT_W8 ? DirectShape{16, 16, 8, 8} : variant == DIRECT_W4 ? DirectShape{16, 16, 4, 4} : variant == DIRECT_COL ? DirectShape{64, 16, 1, 4}
           : DirectShape{32, 32, direct_shared_groups<F>(), 4 * direct_shared_groups<F>()};
}
// All tiles are in one dimension of the grid; outputs beyond it go to the kernels that serve otherwise (posit<8,0>, 131072 x 131072: 2^24 tiles of 512 threads).
inline bool direct_grid_fits(const DirectShape& s, int64_t M, int64_t N) { return ((M + s.tr - 1) / s.tr) * ((N + s.tc - 1) / s.tc) < GRID_THREADS / (64 * s.waves); }

// The fastest way by these estimates, and its us.  posit<32,2> does not have one.
template <class F>
inline DirectPlan direct_plan(int64_t M, int64_t N, int64_t K, double* us) {
    DirectPlan best{DIRECT_NONE, 1, (int)K, 0};
    *us = 1e30;
    if (F::N > 16 || M < 1 || N < 1 || K < 1 || M > ((int64_t)1 << 30) || N > ((int64_t)1 << 20) || K >= ((int64_t)1 << 31)) return best;
    const DirectCost* cost = direct_cost<F>();
    const int64_t nkb = (K + 63) / 64;
    auto estimate = [&](const DirectCost& c, int tr, int tc, int kg, int64_t kb, int64_t slices) {
        const double tiles = (double)((M + tr - 1) / tr) * (double)((N + tc - 1) / tc);
        return c.base + c.unit * tiles * (double)nkb * 1e-3 + c.step * (double)((kb + kg - 1) / kg) + c.group * tiles * (double)slices * 1e-3;
    };
    if (K <= DIRECT_MAXK) {
        for (int v = 0; v < 4; ++v) {
            const DirectShape s = direct_shape<F>(DIRECT_W8 + v);
            const double t = estimate(cost[v], s.tr, s.tc, s.kg, nkb, 1);
            if (t < *us && direct_grid_fits(s, M, N)) {
                *us = t;
                best.variant = DIRECT_W8 + v;
            }
        }
    }
    if (M * N <= 65536) {  // slices of 128 reduction indices and more: their partial quires stay within 26 MB
        for (int s = 4; s <= 16; s *= 2) {
            const int64_t kps = ((K + s - 1) / s + 63) / 64 * 64, slices = (K + kps - 1) / kps;
            if (kps < 128 || kps > DIRECT_MAXK) continue;
            const double t = estimate(cost[DIRECT_SLICED], 16, 16, 8, kps / 64, slices) + 0.5;
            if (t < *us && slices > 1) {
                *us = t;
                best = DirectPlan{DIRECT_W8, (int)slices, (int)kps, (size_t)slices * ((size_t)M * N * Arith<F>::L + M + N) * sizeof(uint32_t)};
            }
        }
    }
    return best;
}

// Whether an estimate (us) is enough below the other kernels'.  It falls behind as products grow: a tenth too long at 2^25 multiply-adds, a fifth too short at 2^28 and
// more, where rounds of workgroups and the operands' second reading from the caches count.  981 products of (8,1), (8,2), (10,1), (12,1) and posit<16,1>, 2^24 to 2^29.5,
// timed on both: 16 chosen with a loss of more than 3 % (without this correction and a margin of 8 %, 20 % for (8,1), 42: (10,1) 4560 x 416 x 224 25 us
// prepared and 34 direct, (12,1) 5431 x 151 x 104 19.4 and 23.3), a mean of 1.4 % lost to the better choice.
inline bool direct_pays(double us, double macs, double other) { return us * (1 + 0.3 * macs / (1 << 30)) < 0.88 * other; }

// Whether the operands lie within what the kernel's offsets reach; pitches are not known to the plan.
inline bool direct_extent_fits(int transA, int transB, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t elem) {
    const int64_t a = (transA ? K : M), b = (transB ? N : K), most = DIRECT_EXTENT / elem;
    return a <= most / (lda > 0 ? lda : 1) && b <= most / (ldb > 0 ? ldb : 1);
}

// posit<32,2> without a bias
hipError_t launch_direct_p32(hipStream_t st, int transA, int transB, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                             void* C, int64_t ldc, int fout);

template <class F>
hipError_t launch_direct_gemm(hipStream_t st, const DirectPlan& p, int transA, int transB, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
                              const void* B, int64_t ldb, const void* bias, void* C, int64_t ldc, int fout, void* workspace);

}  // namespace pnn
