// The three passes of a convolution layer on direct_kernel (direct_mfma.h).
#include "direct_conv.h"

#include "direct_mfma.h"

namespace pnn {

// Forward, left operand: row = (n, oh, ow), k = (c, r, s).  The indices of 16 consecutive k are stepped, not divided.
template <class T>
struct DirectConvX {
    static constexpr bool RAISES_NAR = true;
    const T* x;
    ConvGeom g;
    int rows;
    struct Row { uint32_t image; int ih, iw; };  // element (n, 0, 0, 0); where tap (0, 0) reads
    __device__ __forceinline__ Row row(int r) const {
        r = r < rows ? r : rows - 1;
        const int ohw = g.OH * g.OW, n = r / ohw, rem = r - n * ohw, oh = rem / g.OW;
        return Row{(uint32_t)n * (uint32_t)(g.C * g.H * g.W), oh * g.sh - g.ph, (rem - oh * g.OW) * g.sw - g.pw};
    }
    __device__ __forceinline__ void fetch(const Row& q, int k0, int kend, DirectRaw<T>& raw) const {
        const int rs = g.R * g.S;
        int c = k0 / rs, r = (k0 - c * rs) / g.S, s = k0 - c * rs - r * g.S;
        raw.gather([&](int i) {
            const int ih = q.ih + r, iw = q.iw + s;
            const bool in = (k0 + i < kend) & ((unsigned)ih < (unsigned)g.H) & ((unsigned)iw < (unsigned)g.W);
            const uint32_t at = in ? q.image + (uint32_t)((c * g.H + ih) * g.W + iw) : 0u;
            const T v = *(const T*)((const char*)x + at * (uint32_t)sizeof(T));
            if (++s == g.S) {
                s = 0;
                if (++r == g.R) {
                    r = 0;
                    ++c;
                }
            }
            return in ? v : (T)0;
        });
    }
};

// Backward-data, left operand: row = (n, h, w), k = (ko, r, s) -> dy[n, ko, (h + ph - r) / sh, (w + pw - s) / sw] where that is whole
template <class T>
struct DirectConvDy {
    static constexpr bool RAISES_NAR = true;
    const T* dy;
    ConvGeom g;
    int rows;
    uint32_t div_h, div_w;  // floor(2^32 / stride) + 1; strides above 1
    struct Row { uint32_t image; int th, tw; };
    __device__ __forceinline__ Row row(int r) const {
        r = r < rows ? r : rows - 1;
        const int hw = g.H * g.W, n = r / hw, rem = r - n * hw, h = rem / g.W;
        return Row{(uint32_t)n * (uint32_t)(g.K * g.OH * g.OW), h + g.ph, rem - h * g.W + g.pw};
    }
    __device__ __forceinline__ void fetch(const Row& q, int k0, int kend, DirectRaw<T>& raw) const {
        const int rs = g.R * g.S;
        int c = k0 / rs, r = (k0 - c * rs) / g.S, s = k0 - c * rs - r * g.S;
        const bool strided = g.sh != 1 || g.sw != 1;
        raw.gather([&](int i) {
            const int th = q.th - r, tw = q.tw - s;
            int oh = th, ow = tw;
            bool in = (k0 + i < kend) & (th >= 0) & (tw >= 0);
            if (strided) {  // exact below 2^16, as direct_conv_plan sees to
                if (g.sh != 1) oh = (int)__umulhi((uint32_t)th, div_h);
                if (g.sw != 1) ow = (int)__umulhi((uint32_t)tw, div_w);
                in &= (oh * g.sh == th) & (ow * g.sw == tw);
            }
            in &= (oh < g.OH) & (ow < g.OW);
            const uint32_t at = in ? q.image + (uint32_t)((c * g.OH + oh) * g.OW + ow) : 0u;
            const T v = *(const T*)((const char*)dy + at * (uint32_t)sizeof(T));
            if (++s == g.S) {
                s = 0;
                if (++r == g.R) {
                    r = 0;
                    ++c;
                }
            }
            return in ? v : (T)0;
        });
    }
};

// Backward-data, right operand: row = c, k = (ko, r, s) -> w[ko, c, r, s]; NaR counts as zero (bwd_data_nar_weights_kernel)
template <class T>
struct DirectConvW {
    static constexpr bool RAISES_NAR = false;
    const T* w;
    int rs, step, rows;  // step: elements from the last tap of (ko, c) to the first of (ko + 1, c)
    typedef int Row;
    __device__ __forceinline__ Row row(int r) const { return r < rows ? r : rows - 1; }
    __device__ __forceinline__ void fetch(Row c, int k0, int kend, DirectRaw<T>& raw) const {
        const int ko = k0 / rs;
        int t = k0 - ko * rs;
        uint32_t at = (uint32_t)(ko * rows + c) * (uint32_t)rs + (uint32_t)t;
        raw.gather([&](int i) {
            const bool in = k0 + i < kend;
            const T v = *(const T*)((const char*)w + (in ? at : 0u) * (uint32_t)sizeof(T));
            ++at;
            if (++t == rs) {
                t = 0;
                at += (uint32_t)step;
            }
            return in ? v : (T)0;
        });
    }
};

// Backward-weight, left operand: row = ko, k = (n, oh, ow) -> dy[n, ko, oh, ow]
template <class T>
struct DirectConvDyRows {
    static constexpr bool RAISES_NAR = true;
    const T* dy;
    int ohw, rows;
    typedef int Row;
    __device__ __forceinline__ Row row(int r) const { return r < rows ? r : rows - 1; }
    __device__ __forceinline__ void fetch(Row ko, int k0, int kend, DirectRaw<T>& raw) const {
        const int n = k0 / ohw;
        int p = k0 - n * ohw;
        uint32_t at = (uint32_t)(n * rows + ko) * (uint32_t)ohw + (uint32_t)p;
        if (p + 16 <= ohw && k0 + 16 <= kend) {
            __builtin_memcpy(raw.w, (const char*)dy + at * (uint32_t)sizeof(T), 16 * sizeof(T));  // any alignment
            return;
        }
        raw.gather([&](int i) {
            const bool in = k0 + i < kend;
            const T v = *(const T*)((const char*)dy + (in ? at : 0u) * (uint32_t)sizeof(T));
            ++at;
            if (++p == ohw) {
                p = 0;
                at += (uint32_t)(rows - 1) * (uint32_t)ohw;
            }
            return in ? v : (T)0;
        });
    }
};

// Backward-weight, right operand: row = (c, r, s), k = (n, oh, ow) -> x[n, c, oh sh + r - ph, ow sw + s - pw]; row C R S: ones
template <class T>
struct DirectConvXCols {
    static constexpr bool RAISES_NAR = true;
    const T* x;
    ConvGeom g;
    int crs;
    uint32_t one;
    struct Row { uint32_t plane; int dr, ds; };  // element (0, c, 0, 0)
    __device__ __forceinline__ Row row(int i) const {
        if (i >= crs) return Row{0u, 0, i == crs ? 0x10000 : 0x20000};  // the ones; beyond them anything
        const int rs = g.R * g.S, c = i / rs, t = i - c * rs, r = t / g.S;
        return Row{(uint32_t)(c * g.H * g.W), r - g.ph, t - r * g.S - g.pw};
    }
    __device__ __forceinline__ void fetch(const Row& q, int k0, int kend, DirectRaw<T>& raw) const {
        const int ohw = g.OH * g.OW;
        int n = k0 / ohw, oh = (k0 - n * ohw) / g.OW, ow = k0 - n * ohw - oh * g.OW;
        const uint32_t image = (uint32_t)(g.C * g.H * g.W);
        uint32_t base = (uint32_t)n * image + q.plane;
        const T other = q.ds == 0x10000 ? (T)one : (T)0;
        raw.gather([&](int i) {
            const int ih = oh * g.sh + q.dr, iw = ow * g.sw + q.ds;
            const bool live = k0 + i < kend, in = live & ((unsigned)ih < (unsigned)g.H) & ((unsigned)iw < (unsigned)g.W);
            const T v = *(const T*)((const char*)x + (in ? base + (uint32_t)(ih * g.W + iw) : 0u) * (uint32_t)sizeof(T));
            if (++ow == g.OW) {
                ow = 0;
                if (++oh == g.OH) {
                    oh = 0;
                    base += image;
                }
            }
            return in ? v : live ? other : (T)0;
        });
    }
};

template <class F>
hipError_t launch_direct_conv(hipStream_t st, const DirectConvPlan& p, const ConvGeom& g, const void* a, const void* b, const void* bias, void* out, void* dbias,
                              int fout, void* workspace) {
    typedef typename Storage<F::N>::T T;
    const int M = p.M, N = p.N, K = p.K;
    if (p.which == 0) {
        const DirectConvX<T> x{(const T*)a, g, M};
        const DirectMatrix<T> w{(const T*)b, (uint32_t)K * (uint32_t)sizeof(T), (uint32_t)sizeof(T), N};
        return launch_direct<F>(st, p.cut, x, w, NchwOut{(int64_t)g.OH * g.OW, (int64_t)g.K}, M, N, K, bias, out, fout, workspace);
    }
    if (p.which == 1) {
        auto magic = [](int d) { return d > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)d) + 1u : 0u; };
        const DirectConvDy<T> dy{(const T*)a, g, M, magic(g.sh), magic(g.sw)};
        const DirectConvW<T> w{(const T*)b, g.R * g.S, (g.C - 1) * g.R * g.S, g.C};
        return launch_direct<F>(st, p.cut, dy, w, NchwOut{(int64_t)g.H * g.W, (int64_t)g.C}, M, N, K, nullptr, out, fout, workspace);
    }
    const int crs = g.C * g.R * g.S;
    const DirectConvDyRows<T> dy{(const T*)a, g.OH * g.OW, g.K};
    const DirectConvXCols<T> x{(const T*)b, g, crs, F::NAR >> 1};
    return launch_direct<F>(st, p.cut, dy, x, WeightAndBiasOut{crs, dbias}, M, N, K, nullptr, out, fout, workspace);
}

#define PNN_DIRECT_CONV(F)                                                                                                                             \
    template hipError_t launch_direct_conv<F>(hipStream_t, const DirectConvPlan&, const ConvGeom&, const void*, const void*, const void*, void*, void*, int, \
                                              void*);
PNN_DIRECT_CONV(P8)
PNN_DIRECT_CONV(P8_1)
PNN_DIRECT_CONV(P8_2)
PNN_DIRECT_CONV(P10_1)
PNN_DIRECT_CONV(P10_2)
PNN_DIRECT_CONV(P12_1)
PNN_DIRECT_CONV(P12_2)
PNN_DIRECT_CONV(P16)

}  // namespace pnn
