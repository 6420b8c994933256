// Which convolutions take direct_kernel (direct_mfma.h), how they are cut, and their launch (direct_conv.hip).
#pragma once

#include "conv_b8.h"
#include "conv_desc.h"
#include "conv_dig_mfma.h"
#include "conv_p8_mfma.h"
#include "direct_gemm.h"

namespace pnn {

// us of a pass.  Forward and backward-data by the four variants: as DirectCost in direct_gemm.h, and per 10^6 outputs, whose stores are apart by a plane of the image.  The weight
// gradient, 16 x 16 with eight waves: base, sliced base, per 1000 (tile, k block), per k block of a wave, per 1000 (tile, slice), merge per 10^6 partial quires.  Fitted to 10007 layers of
// 2^17 to 2^30 multiply-adds in nine formats, every variant and three numbers of slices timed on each (NaR marking and the gradient of the bias included); off by 7 to 17 % (root
// mean square), up to a third where the last round of workgroups is nearly empty.  The variant chosen by it loses 1.5 % to the best one in the mean.
struct DirectConvPass { float base, unit, step, group, output; };
struct DirectConvCost { DirectConvPass pass[2][4]; float bw[6]; };
template <class F>
inline const DirectConvCost& direct_conv_cost() {
    static const DirectConvCost COST[8] = {
        {{{{2.68f, 0.605f, 1.75f, 4.02f, 2.68f}, {2.97f, 0.683f, 1.63f, 1.34f, 3.49f}, {4.69f, 2.49f, 1.67f, 1.06f, 4.92f}, {2.82f, 1.92f, 2.1f, 2.61f, 4.08f}},  // posit<8,0>
          {{2.72f, 0.837f, 3.21f, 5.19f, 0.f}, {3.7f, 0.928f, 2.41f, 1.85f, 2.39f}, {5.26f, 3.41f, 2.4f, 1.32f, 3.75f}, {3.88f, 2.76f, 2.44f, 5.19f, 2.91f}}},
         {3.9f, 6.65f, 0.843f, 1.61f, 2.81f, 3.8f}},
        {{{{2.65f, 0.622f, 2.f, 6.61f, 2.17f}, {3.28f, 0.692f, 1.73f, 2.26f, 4.07f}, {5.44f, 2.74f, 1.71f, 1.f, 6.09f}, {3.09f, 2.69f, 2.18f, 4.63f, 5.07f}},  // (8,1)
          {{2.74f, 0.906f, 3.31f, 7.43f, 1.79f}, {3.88f, 0.961f, 2.54f, 3.29f, 2.84f}, {5.98f, 3.74f, 2.4f, 1.49f, 4.99f}, {4.47f, 3.11f, 2.53f, 5.47f, 4.68f}}},
         {4.63f, 7.24f, 1.f, 1.53f, 3.31f, 6.65f}},
        {{{{2.9f, 1.07f, 2.03f, 12.7f, 5.46f}, {3.24f, 0.915f, 1.99f, 4.36f, 7.51f}, {5.98f, 3.32f, 2.01f, 1.75f, 12.2f}, {2.85f, 5.11f, 2.93f, 10.6f, 9.87f}},  // (8,2)
          {{2.69f, 1.38f, 3.59f, 15.8f, 2.39f}, {4.1f, 1.19f, 2.77f, 5.22f, 5.56f}, {6.6f, 4.63f, 2.75f, 3.1f, 8.88f}, {4.02f, 5.82f, 3.17f, 12.7f, 8.69f}}},
         {4.77f, 7.79f, 1.5f, 1.63f, 6.84f, 12.f}},
        {{{{2.56f, 0.768f, 2.64f, 7.67f, 6.86f}, {3.23f, 0.828f, 2.21f, 3.13f, 7.19f}, {6.11f, 3.21f, 2.09f, 0.568f, 10.f}, {3.38f, 3.31f, 2.52f, 4.39f, 7.92f}},  // (10,1)
          {{3.13f, 1.09f, 3.56f, 8.4f, 6.44f}, {3.98f, 1.16f, 2.68f, 5.06f, 5.2f}, {6.59f, 4.38f, 2.68f, 2.16f, 6.36f}, {4.69f, 3.5f, 2.79f, 6.43f, 5.78f}}},
         {4.76f, 7.85f, 1.18f, 1.63f, 4.72f, 2.9f}},
        {{{{2.7f, 0.898f, 2.64f, 8.87f, 7.72f}, {3.55f, 0.931f, 2.16f, 5.71f, 7.46f}, {5.84f, 4.08f, 1.9f, 4.59f, 12.4f}, {2.97f, 4.91f, 2.57f, 11.f, 10.6f}},  // (12,1)
          {{3.23f, 1.13f, 3.81f, 9.93f, 6.8f}, {4.36f, 1.21f, 3.07f, 6.37f, 6.5f}, {6.9f, 5.54f, 2.63f, 5.68f, 9.27f}, {4.11f, 5.77f, 3.17f, 12.8f, 9.54f}}},
         {5.35f, 8.22f, 1.22f, 1.79f, 4.62f, 12.7f}},
        {{{{2.88f, 1.39f, 2.58f, 18.3f, 13.2f}, {3.13f, 1.21f, 2.56f, 9.43f, 9.77f}, {6.63f, 4.63f, 2.55f, 6.26f, 16.6f}, {4.68f, 9.25f, 2.63f, 12.f, 24.5f}},  // (10,2)
          {{2.8f, 1.73f, 3.84f, 19.1f, 15.8f}, {4.06f, 1.58f, 3.19f, 10.f, 9.68f}, {7.35f, 6.67f, 3.17f, 5.91f, 12.9f}, {5.55f, 11.1f, 2.93f, 12.7f, 19.7f}}},
         {5.59f, 8.23f, 1.74f, 1.84f, 11.2f, 16.3f}},
        {{{{2.55f, 1.55f, 3.71f, 22.f, 12.1f}, {3.36f, 2.24f, 2.86f, 23.5f, 11.2f}, {7.21f, 9.52f, 2.47f, 15.9f, 25.7f}, {5.74f, 10.4f, 2.69f, 15.2f, 24.3f}},  // (12,2)
          {{3.2f, 1.88f, 4.36f, 24.1f, 11.1f}, {4.58f, 3.f, 3.29f, 25.f, 10.7f}, {7.52f, 12.3f, 3.45f, 14.5f, 23.9f}, {6.45f, 12.4f, 3.46f, 17.2f, 21.f}}},
         {7.53f, 9.4f, 2.06f, 2.05f, 16.4f, 10.5f}},
        {{{{0.359f, 2.12f, 5.52f, 17.f, 3.75f}, {2.44f, 2.f, 3.42f, 9.23f, 6.05f}, {5.63f, 8.29f, 3.18f, 3.74f, 12.4f}, {2.35f, 7.21f, 3.87f, 12.3f, 10.2f}},  // posit<16,1>
          {{1.77f, 2.45f, 5.54f, 19.2f, 4.44f}, {3.82f, 2.38f, 3.77f, 9.66f, 6.81f}, {6.32f, 10.1f, 3.84f, 3.79f, 9.83f}, {4.13f, 8.5f, 3.93f, 12.4f, 8.54f}}},
         {5.3f, 8.05f, 2.89f, 2.92f, 8.31f, 9.51f}},
    };
    return COST[F::N == 8 ? F::ES : F::ES == 1 ? (F::N == 10 ? 3 : F::N == 12 ? 4 : 7) : F::N == 10 ? 5 : 6];
}

struct DirectConvPlan {
    int which;
    int M, N, K;  // rows, columns, reduction: (n, oh, ow) x k x (c, r, s); (n, h, w) x c x (k, r, s); k x (c, r, s [, ones]) x (n, oh, ow)
    DirectPlan cut;
};

// Offsets are 32 bits, rows and columns of pixels and their products with a stride 16.
inline bool direct_conv_fits(const ConvGeom& g, int64_t elem) {
    const int64_t most = DIRECT_EXTENT / elem, lim = 32767;
    if (g.N <= 0 || g.C <= 0 || g.K <= 0 || g.H > lim || g.W > lim || g.ph > lim || g.pw > lim || g.sh > lim || g.sw > lim || g.R > lim || g.S > lim) return false;
    return (int64_t)g.N * g.C * g.H * g.W <= most && (int64_t)g.N * g.K * g.OH * g.OW <= most && (int64_t)g.K * g.C * g.R * g.S <= most;
}

// The fastest cut of a pass by these estimates, and its us.
template <class F>
inline DirectConvPlan direct_conv_cut(int which, const ConvGeom& g, bool with_bias, double* us) {
    const ConvDims d = conv_dims(which, g);
    DirectConvPlan p{which, (int)d.M, (int)d.N + (which == 2 && with_bias ? 1 : 0), (int)d.K, {DIRECT_NONE, 1, (int)d.K, 0}};
    *us = 1e30;
    if (F::N > 16 || d.M < 1 || d.N < 1 || d.K < 1 || d.N > ((int64_t)1 << 20) || !direct_conv_fits(g, F::N == 8 ? 1 : 2)) return p;
    const DirectConvCost& cost = direct_conv_cost<F>();
    const double nkb = (double)((d.K + 63) / 64);
    auto tiles = [&](int tr, int tc) { return 1e-3 * (double)((p.M + tr - 1) / tr) * (double)((p.N + tc - 1) / tc); };
    if (which < 2) {
        if (d.K > DIRECT_MAXK) return p;
        for (int v = 0; v < 4; ++v) {
            const DirectShape s = direct_shape<F>(DIRECT_W8 + v);
            const DirectConvPass& c = cost.pass[which][v];
            const double n = tiles(s.tr, s.tc), t = c.base + (c.unit * nkb + c.group) * n + c.step * (double)(((int64_t)nkb + s.kg - 1) / s.kg) + c.output * 1e-6 * p.M * p.N;
            if (t < *us && direct_grid_fits(s, d.M, d.N)) {
                *us = t;
                p.cut.variant = DIRECT_W8 + v;
            }
        }
        return p;
    }
    const double n = tiles(16, 16);
    if (!direct_grid_fits(direct_shape<F>(DIRECT_W8), p.M, p.N)) return p;
    for (int64_t s = 1; s <= 256; s *= 2) {
        const int64_t kps = s == 1 ? d.K : ((d.K + s - 1) / s + 63) / 64 * 64, slices = (d.K + kps - 1) / kps;
        const size_t bytes = slices > 1 ? (size_t)slices * ((size_t)p.M * p.N * Arith<F>::L + p.M + p.N) * sizeof(uint32_t) : 0;
        if (kps > DIRECT_MAXK || bytes > ((size_t)64 << 20) || (s > 1 && slices == 1)) continue;
        const double t = cost.bw[slices > 1 ? 1 : 0] + (cost.bw[2] * nkb + cost.bw[4] * (double)slices) * n + cost.bw[3] * (double)((kps + 511) / 512) +
                         (slices > 1 ? cost.bw[5] * 1e-6 * (double)slices * p.M * p.N : 0);
        if (t < *us) {
            *us = t;
            p.cut = DirectPlan{DIRECT_W8, (int)slices, (int)kps, bytes};
        }
    }
    return p;
}

// Most outputs of a forward or backward-data pass with a reduction of up to half a k block, where the general kernel serves it otherwise (see direct_short_outputs; gathered
// operands cost this kernel more).  us, general and direct: 1 x 1 forward, (12,2), 158 images of 9 channels at 40 x 40 to 54 541 and 784, 285 of 4 at 35 x 35 to 52, stride 2,
// 164 and 271; backward-data, stride 2, posit<8,0>, 190 of 98 at 37 x 37 to 7 132 and 243, posit<16,1>, 12 of 81 at 53 x 53 to 4 68 and 87; (12,2), 14 of 50 at 39 x 39 to 5
// 59 and 77; 5 of 104 at 55 x 55 to 13, (10,2), 51 and 53.  Below, of 590 timed passes, two were more than 3 % behind.
constexpr double CONV_GENERAL_US = 1e9;
template <class F>
constexpr int64_t direct_conv_short_outputs(int64_t K) {
    constexpr bool longest = F::N == 12 && F::ES == 2;  // eleven planes
    if (K > 32) return INT64_MAX;
    if (K <= 16) return (int64_t)1 << (longest ? 18 : 19);
    return longest ? (int64_t)1 << 19 : F::N == 10 ? INT64_MAX : (int64_t)1 << 22;
}

// us of the kernels that take a pass otherwise: rewritten operands on the matrix cores (fitted to 90 to 1910 layers each, off by 7 to 13 %), the
// byte gather of (8,1) and (8,2), the dot products of posit<8,0> (15 to 30 %).  The general kernel, a tenth of their rate and less: CONV_GENERAL_US.
// planes: whether it is the first of these.
template <class F>
inline double conv_prepared_us(int which, const ConvGeom& g, bool with_bias, bool* planes_serve = nullptr) {
    constexpr bool p8 = F::N == 8 && F::ES == 0;
    const ConvDims d = conv_dims(which, g);
    const double P = (double)(which == 2 ? d.K : d.M);
    if (which == 2) {
        bool planes = false;
        if (p8) planes = p8_conv_eligible(2, g) && p8_conv_bw_plan(g, with_bias).ok;
        else if constexpr (dig_conv_format<F>()) planes = dig_conv_bw_plan<F>(g, with_bias).ok;
        if (planes_serve) *planes_serve = planes;
        if (planes) {  // launches, the rewritten operands, the products of whole tiles
            const int ng = (g.N + 15) / 16, wy = g.K > 32 ? 2 : 1, tr = 32 * wy, tc = (p8 ? 128 : 64) / wy;
            const double rows = (double)((g.K + tr - 1) / tr) * tr, cols = (double)((d.N + with_bias + tc - 1) / tc) * tc, k = 16.0 * g.OH * g.OW * ng;
            const double mb = ((double)g.C * g.H * g.W * ng * 16 + k * rows) / (1 << 20), work = 1e-9 * k * rows * cols;
            return p8 ? 19.3 + 0.561 * mb + 9.5 * work : F::N == 8 ? (F::ES == 1 ? 25 + 1.07 * mb : 28.2 + 1.21 * mb) + 16.2 * work : 27.3 + 1.88 * mb + 16.2 * work;
        }
        if constexpr (F::N == 8 && F::ES != 0) {
            if (p8_conv_eligible(2, g)) return b8_conv_us<F>(true, (int)d.N, g.K, (int)d.K) - (with_bias ? 0.0 : 8.0);
        }
        return p8 && p8_conv_eligible(2, g) ? 28.8 + 0.0457 * P : CONV_GENERAL_US;
    }
    bool planes = false;
    if (p8) planes = p8_conv_eligible(which, g) && p8_conv_mfma_plan(which, g).ok;
    else if constexpr (dig_conv_format<F>()) planes = dig_conv_plan<F>(which, g).ok;
    if (planes_serve) *planes_serve = planes;
    if (planes) {  // launches, a workgroup's k blocks, the rounds of workgroups behind the first, the rewritten tensor, the outputs
        const int ci = which == 0 ? g.C : g.K, mo = which == 0 ? g.K : g.C, wy = mo > 32 ? 2 : 1, tc = (p8 ? 128 : 64) / wy, cg = (ci + 15) / 16;
        const double kb = (double)(((int64_t)g.R * g.S * cg + 1) / 2), pixels = which == 0 ? (double)g.N * g.H * g.W : (double)g.N * g.OH * g.OW;
        const double groups = (double)((mo + 32 * wy - 1) / (32 * wy)) * (double)(((int64_t)d.M + tc - 1) / tc), at_once = p8 ? 256 : kb <= 8 || groups > 768 ? 1024 : 768;
        const double rounds = groups > at_once ? groups / at_once - 1 : 0, mb = pixels * cg * 16 / (1 << 20), out = (double)d.M * mo * (F::N == 8 ? 1 : 2) / (1 << 20);
        static const float C[4][2][6] = {{{7.88f, 0.481f, 0.148f, 0.711f, 1.01f, 0.f}, {8.85f, 0.513f, 0.166f, 0.651f, 1.f, 0.f}},
                                         {{15.1f, 0.48f, 0.615f, 3.03f, 2.77f, 1.71f}, {14.4f, 0.396f, 0.686f, 1.93f, 3.23f, 1.31f}},
                                         {{17.4f, 0.401f, 0.716f, 2.96f, 3.09f, 1.6f}, {15.f, 0.438f, 0.648f, 2.59f, 3.46f, 1.45f}},
                                         {{16.1f, 0.439f, 0.633f, 4.02f, 3.04f, 1.01f}, {15.f, 0.387f, 0.671f, 2.89f, 3.45f, 0.825f}}};
        const float* c = C[F::N == 8 ? F::ES : 3][which];
        return c[0] + c[1] * kb + (c[2] * kb + c[3]) * rounds + c[4] * mb + c[5] * out;
    }
    if constexpr (F::N == 8 && F::ES != 0) {
        if (p8_conv_eligible(which, g)) return b8_conv_us<F>(false, (int)d.M, (int)d.N, (int)d.K) + (which == 1 ? 2 : 0);
    }
    if (p8 && p8_conv_eligible(which, g)) {  // one launch where the stride is not one, two with decoded operands
        const double outputs = 1e-6 * P * (double)d.N, macs = 1e-3 * outputs * (double)d.K, k = 1e-3 * (double)d.K;
        return 0.9 * (which == 1 ? 14.8 + 1.9 * outputs + 19 * macs + 29 * k : g.sh == 1 && g.sw == 1 ? 14 + 1.45 * outputs + 49 * macs + 23 * k : 9.3 + 0.58 * outputs + 28.5 * macs + 100 * k);
    }
    return CONV_GENERAL_US;
}

// Layers that go to the matrix cores straight from their patterns: where the estimate is a tenth below the digit planes', a quarter from 60 us on (posit(8,1) forward of 235 images of
// 84 channels at 38 x 38 to 23, 1 x 1, 104 us there, 147 here, estimated 159 and 125), and 15 % below the other kernels', whose estimates are off by more.  Of the 5599 of those 10007 layers that another fast kernel serves, 2969 go direct, 18 of them more than 3 % slower than on that kernel; in the mean
// 2.4 % lost to the better choice.  The formats without planes take 0.2 of the general kernel's time.
template <class F>
inline DirectConvPlan direct_conv_plan(int which, const ConvGeom& g, bool with_bias) {
    double us;
    DirectConvPlan p = direct_conv_cut<F>(which, g, with_bias, &us);
    if (p.cut.variant == DIRECT_NONE) return p;
    bool planes = false;
    const double other = conv_prepared_us<F>(which, g, with_bias, &planes);
    // (posit<8,0> dot products of more than 1500 indices take down to 0.6 of their estimate: forward of 104 images of 65 channels at 8 x 8 to 118, 5 x 5, 62 us, estimated 104; here 81)
    const double least = planes ? (us > 60 ? 0.75 : 0.9) : F::N == 8 && F::ES == 0 && p.K > 1500 ? 0.55 : 0.85;
    if (us >= least * other || (other == CONV_GENERAL_US && (int64_t)p.M * p.N > direct_conv_short_outputs<F>(p.K))) p.cut = DirectPlan{DIRECT_NONE, 1, 0, 0};
    return p;
}

template <class F>
hipError_t launch_direct_conv(hipStream_t st, const DirectConvPlan& p, const ConvGeom& g, const void* a, const void* b, const void* bias, void* out, void* dbias,
                              int fout, void* workspace);

}  // namespace pnn
