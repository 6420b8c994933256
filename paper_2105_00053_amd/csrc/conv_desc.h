// Host-side reading of a pnn_conv2d_desc: validation, output size, and the
// dimensions of the implicit GEMM each of the three passes runs as (paper
// Sec. 3.1: convolution forward, backward-data, backward-weight).
#pragma once

#include "api_common.h"
#include "quire_gemm.h"

namespace pnn {

inline bool conv_geom(const pnn_conv2d_desc* d, ConvGeom* g) {
    if (!d) return false;
    if (d->N < 0 || d->C < 0 || d->H <= 0 || d->W <= 0 || d->K < 0 || d->R <= 0 || d->S <= 0) return false;
    if (d->pad_h < 0 || d->pad_w < 0 || d->stride_h <= 0 || d->stride_w <= 0) return false;
    if (d->H + 2 * d->pad_h < d->R || d->W + 2 * d->pad_w < d->S) return false;
    const int64_t lim = (int64_t)1 << 30;
    if (d->N >= lim || d->C >= lim || d->H >= lim || d->W >= lim || d->K >= lim || d->R >= lim || d->S >= lim) return false;
    g->N = (int)d->N; g->C = (int)d->C; g->H = (int)d->H; g->W = (int)d->W;
    g->K = (int)d->K; g->R = (int)d->R; g->S = (int)d->S;
    g->ph = (int)d->pad_h; g->pw = (int)d->pad_w; g->sh = (int)d->stride_h; g->sw = (int)d->stride_w;
    g->OH = (int)((d->H + 2 * d->pad_h - d->R) / d->stride_h + 1);
    g->OW = (int)((d->W + 2 * d->pad_w - d->S) / d->stride_w + 1);
    // every index the kernels form must fit 31 bits
    if ((int64_t)g->C * g->R * g->S >= lim || (int64_t)g->K * g->R * g->S >= lim) return false;
    if ((int64_t)g->N * g->OH * g->OW >= lim || (int64_t)g->N * g->H * g->W >= lim) return false;
    return true;
}

struct ConvDims {
    int64_t M, N, K;
};

inline ConvDims conv_dims(int which, const ConvGeom& g) {
    ConvDims d;
    if (which == 0) { d.M = (int64_t)g.N * g.OH * g.OW; d.N = g.K; d.K = (int64_t)g.C * g.R * g.S; }
    else if (which == 1) { d.M = (int64_t)g.N * g.H * g.W; d.N = g.C; d.K = (int64_t)g.K * g.R * g.S; }
    else { d.M = g.K; d.N = (int64_t)g.C * g.R * g.S; d.K = (int64_t)g.N * g.OH * g.OW; }
    return d;
}

// The gathering matrix-core kernels keep a tap's row and column offsets in 16 bits, stand -40000 and 0x7FFF rows for "no pixel"
// and form addresses in 32 bits, those of taps in the border included.  Whether that holds where output (oh, ow) of image i
// reads tap (r, s) at input (oh sh + r - offh, ow sw + s - offw), `unit` words per pixel; HI and WI are at most 16384.
inline bool conv_gather_fits(int64_t NI, int64_t HI, int64_t WI, int64_t HO, int64_t WO, int64_t R, int64_t S, int64_t offh, int64_t offw, int64_t sh,
                             int64_t sw, int64_t unit) {
    const int64_t most = 16384, last_h = R - 1 - offh, last_w = S - 1 - offw;
    if (offh > most || offw > most || last_h > most || last_w > most) return false;
    const int64_t far = ((NI - 1) * HI + (HO - 1) * sh) * WI + (WO - 1) * sw, ahead = last_h * WI + last_w, behind = offh * WI + offw;
    return (far + (ahead > 0 ? ahead : 0)) * unit < ((int64_t)1 << 31) && behind * unit < ((int64_t)1 << 31);
}

// Backward-data on digit planes, NaR weights (see bwd_data_nar_weights_kernel, whose launch this replaces: 1.3 us of a call).
// w: the weights, null where nothing is to be marked.  A workgroup marks its own tile, channels c0 .. c0 + TR - 1 and positions
// p0 .. p0 + TC - 1, when everything that stores there has done so; it is called only if the weights hold NaR.
struct BwdDataNar {
    const void* w;  // [K][C][R][S]
    int K, C, R, S, ph, pw, OH, OW, H, W, P;
    FmtRT fin, fout;
};

template <int TR, int TC>
__device__ __forceinline__ void bwd_data_nar_tile(const BwdDataNar& g, void* dx, int c0, int p0) {
    const int rs = g.R * g.S, rows = g.C - c0 < TR ? g.C - c0 : TR;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's own stores of the tile are done
    __syncthreads();                // everyone's are
    for (int64_t i = threadIdx.x; i < (int64_t)rows * g.K * rs; i += 256) {
        const int tap = (int)(i % rs), k = (int)(i / rs % g.K), c = c0 + (int)(i / ((int64_t)rs * g.K));
        const int64_t at = ((int64_t)k * g.C + c) * rs + tap;
        const uint32_t v = g.fin.n <= 8 ? ((const uint8_t*)g.w)[at] : ((const uint16_t*)g.w)[at];
        if (v != g.fin.nar()) continue;
        const int r = tap / g.S, s = tap % g.S;
        for (int p = p0; p < p0 + TC && p < g.P; ++p) {
            const int n = p / (g.H * g.W), rem = p % (g.H * g.W);
            const int oh = rem / g.W + g.ph - r, ow = rem % g.W + g.pw - s;  // unit stride
            if (oh < 0 || oh >= g.OH || ow < 0 || ow >= g.OW) continue;
            const int64_t o = ((int64_t)n * g.C + c) * g.H * g.W + rem;
            if (g.fout.n <= 8) ((uint8_t*)dx)[o] = (uint8_t)g.fout.nar();
            else if (g.fout.n <= 16) ((uint16_t*)dx)[o] = (uint16_t)g.fout.nar();
            else ((uint32_t*)dx)[o] = g.fout.nar();
        }
    }
}

inline BwdDataNar bwd_data_nar(const void* w, int fin, int fout, const ConvGeom& g) {
    return BwdDataNar{w, g.K, g.C, g.R, g.S, g.ph, g.pw, g.OH, g.OW, g.H, g.W, g.N * g.H * g.W, fmt_of_code(fin), fmt_of_code(fout)};
}

}  // namespace pnn
