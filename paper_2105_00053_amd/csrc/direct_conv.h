// Which convolutions take direct_kernel (direct_mfma.h), how they are cut, and their launch (direct_conv.hip).
#pragma once

#include "conv_b8.h"
#include "conv_desc.h"
#include "conv_dig_mfma.h"
#include "conv_p8_mfma.h"
#include "direct_gemm.h"

namespace pnn {

// us of a pass: forward and backward-data by the four variants, as DirectCost in direct_gemm.h; the weight gradient, 16 x 16 with eight waves: sliced
// base, base, unit, step, group, and merge per 10^6 partial quires.  Fitted to 250 layers per format of 2^17 to 2^29 multiply-adds (NaR
// marking and the gradient of the bias included); off by 8 to 16 %.  Rows: posit<8,0>, (8,1), (8,2), (10,1) and (12,1), the others.
struct DirectConvCost { DirectCost pass[2][4]; float bw[6]; };
template <class F>
inline const DirectConvCost& direct_conv_cost() {
    static const DirectConvCost COST[5] = {
        {{{{3.79f, 0.401f, 2.95f, 4.41f}, {6.03f, 0.589f, 0.901f, 1.85f}, {6.38f, 2.08f, 1.41f, 4.69f}, {5.47f, 1.64f, 1.61f, 4.56f}},
          {{7.55f, 0.73f, 1.72f, 4.68f}, {8.3f, 0.849f, 1.51f, 1.85f}, {8.27f, 3.11f, 1.86f, 3.18f}, {7.9f, 2.72f, 1.54f, 5.08f}}},
         {9.35f, 6.36f, 0.49f, 1.9f, 3.73f, 2.24f}},
        {{{{3.13f, 0.552f, 2.85f, 6.8f}, {4.71f, 0.651f, 1.55f, 2.88f}, {6.43f, 2.24f, 1.59f, 5.94f}, {4.73f, 2.49f, 1.85f, 7.18f}},
          {{6.49f, 0.848f, 2.09f, 7.25f}, {6.99f, 0.933f, 1.92f, 3.37f}, {7.57f, 3.3f, 2.16f, 4.82f}, {7.14f, 3.02f, 2.01f, 6.66f}}},
         {8.84f, 6.01f, 0.512f, 2.2f, 6.07f, 3.98f}},
        {{{{1.8f, 0.848f, 3.7f, 14.1f}, {4.52f, 0.806f, 1.65f, 5.84f}, {7.28f, 2.68f, 1.75f, 10.8f}, {3.7f, 4.88f, 2.29f, 15.4f}},
          {{6.01f, 1.33f, 1.97f, 15.7f}, {6.37f, 1.15f, 2.34f, 5.67f}, {7.79f, 3.93f, 2.46f, 8.57f}, {5.75f, 6.11f, 2.41f, 14.7f}}},
         {7.99f, 5.36f, 0.652f, 2.69f, 15.2f, 2.83f}},
        {{{{2.68f, 0.755f, 3.3f, 10.3f}, {4.43f, 0.741f, 2.02f, 7.2f}, {7.34f, 3.06f, 1.59f, 13.8f}, {4.04f, 4.57f, 2.12f, 16.3f}},
          {{5.33f, 1.07f, 2.99f, 10.5f}, {5.82f, 1.19f, 2.69f, 7.08f}, {7.69f, 4.47f, 2.34f, 12.1f}, {5.83f, 5.85f, 2.35f, 15.4f}}},
         {8.35f, 5.74f, 0.692f, 2.83f, 9.f, 4.54f}},
        {{{{0.5f, 1.78f, 6.73f, 18.2f}, {2.85f, 1.84f, 3.23f, 10.5f}, {7.22f, 6.82f, 2.68f, 13.4f}, {3.35f, 7.13f, 3.08f, 16.6f}},
          {{2.61f, 2.43f, 4.72f, 19.7f}, {4.34f, 2.22f, 3.75f, 11.1f}, {7.16f, 8.52f, 3.49f, 11.6f}, {5.03f, 8.45f, 3.27f, 15.1f}}},
         {6.12f, 4.6f, 1.44f, 5.09f, 18.8f, 4.72f}},
    };
    return COST[F::N == 8 ? F::ES : F::ES == 1 && F::N <= 12 ? 3 : 4];
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
            const DirectCost& c = cost.pass[which][v];
            const double n = tiles(s.tr, s.tc), t = c.base + (c.unit * nkb + c.group) * n + c.step * (double)(((int64_t)nkb + s.kg - 1) / s.kg);
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
        const double t = cost.bw[slices > 1 ? 0 : 1] + (cost.bw[2] * nkb + cost.bw[4] * (double)slices) * n + cost.bw[3] * (double)((kps + 511) / 512) +
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

// us of the kernels that take a pass otherwise: rewritten operands on the matrix cores (fitted to 23 to 58 layers each, off by 6 to 14 %), the
// byte gather of (8,1) and (8,2), the dot products of posit<8,0> (12 to 25 %, hence a tenth less).  The general kernel, a tenth of their rate and less: CONV_GENERAL_US.
template <class F>
inline double conv_prepared_us(int which, const ConvGeom& g, bool with_bias) {
    constexpr bool p8 = F::N == 8 && F::ES == 0;
    const ConvDims d = conv_dims(which, g);
    const double P = (double)(which == 2 ? d.K : d.M);
    if (which == 2) {
        bool planes = false;
        if (p8) planes = p8_conv_eligible(2, g) && p8_conv_bw_plan(g, with_bias).ok;
        else if constexpr (dig_conv_format<F>()) planes = dig_conv_bw_plan<F>(g, with_bias).ok;
        if (planes) {
            const int ng = (g.N + 15) / 16, wy = g.K > 32 ? 2 : 1, tr = 32 * wy, tc = 32 * (4 / wy);
            const double rows = (double)((g.K + tr - 1) / tr) * tr, cols = (double)((d.N + with_bias + tc - 1) / tc) * tc, k = 16.0 * g.OH * g.OW * ng;
            const double mb = ((double)g.C * g.H * g.W * ng * 16 + k * rows) / (1 << 20), work = 1e-9 * k * rows * cols;
            return p8 ? 20.1 + 0.49 * mb + 10 * work : F::N == 8 ? (F::ES == 1 ? 28.6 : 32.1) + 0.89 * mb + 17.4 * work : 31.6 + 1.5 * mb + 18 * work;
        }
        if constexpr (F::N == 8 && F::ES != 0) {
            if (p8_conv_eligible(2, g)) return b8_conv_us<F>(true, (int)d.N, g.K, (int)d.K) - (with_bias ? 0.0 : 8.0);
        }
        return p8 && p8_conv_eligible(2, g) ? 20 + 1e-9 * 60 * (double)d.M * (double)d.N * P : CONV_GENERAL_US;
    }
    bool planes = false;
    if (p8) planes = p8_conv_eligible(which, g) && p8_conv_mfma_plan(which, g).ok;
    else if constexpr (dig_conv_format<F>()) planes = dig_conv_plan<F>(which, g).ok;
    if (planes) {
        const int ci = which == 0 ? g.C : g.K, mo = which == 0 ? g.K : g.C, wy = mo > 32 ? 2 : 1, tc = 32 * (4 / wy), cg = (ci + 15) / 16;
        const double groups = (double)((mo + 32 * wy - 1) / (32 * wy)) * (double)(((int64_t)d.M + tc - 1) / tc), waves = groups > 256 ? groups / 256 - 1 : 0;
        const double kb = (double)(((int64_t)g.R * g.S * cg + 1) / 2), pixels = which == 0 ? (double)g.N * g.H * g.W : (double)g.N * g.OH * g.OW;
        const double mb = pixels * cg * 16 / (1 << 20);
        static const float C[3][2][5] = {{{9.5f, 0.48f, 0.128f, 1.f, 0.63f}, {10.8f, 0.45f, 0.1f, 1.3f, 0.73f}},
                                         {{17.f, 0.79f, 0.41f, 2.2f, 2.7f}, {13.7f, 0.81f, 0.39f, 3.7f, 1.5f}},
                                         {{18.5f, 0.78f, 0.39f, 2.7f, 3.3f}, {16.6f, 0.76f, 0.38f, 4.2f, 1.8f}}};
        const float* c = C[p8 ? 0 : F::N == 8 ? 1 : 2][which];
        return c[0] + (F::N == 8 && F::ES == 2 ? 2 : 0) + c[1] * kb + c[2] * kb * waves + c[3] * mb + c[4] * waves;
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

// Layers that go to the matrix cores straight from their patterns.  Against the kernels that serve otherwise, 980 passes of 2^17 to 2^29
// multiply-adds over nine formats: 0.51 of their time in the geometric mean ((10,1) to (12,2) 0.22, 196 of posit<8,0> 0.61).  direct_pays, as for products: of 1800 passes timed
// on all kernels 1414 go direct, 7 of these more than 3 % slower than before there was this kernel (with an uncorrected estimate a tenth below the other 13, up to 21 %: posit(10,1)
// backward-weight of 196 images of 50 channels at 34 x 34 to 8, 3 x 3, 110 us and 133).
template <class F>
inline DirectConvPlan direct_conv_plan(int which, const ConvGeom& g, bool with_bias) {
    double us;
    DirectConvPlan p = direct_conv_cut<F>(which, g, with_bias, &us);
    if (p.cut.variant == DIRECT_NONE) return p;
    const double other = conv_prepared_us<F>(which, g, with_bias);
    if (!direct_pays(us, (double)p.M * (double)p.N * (double)p.K, other) || (other == CONV_GENERAL_US && (int64_t)p.M * p.N > direct_conv_short_outputs<F>(p.K))) p.cut = DirectPlan{DIRECT_NONE, 1, 0, 0};
    return p;
}

template <class F>
hipError_t launch_direct_conv(hipStream_t st, const DirectConvPlan& p, const ConvGeom& g, const void* a, const void* b, const void* bias, void* out, void* dbias,
                              int fout, void* workspace);

}  // namespace pnn
