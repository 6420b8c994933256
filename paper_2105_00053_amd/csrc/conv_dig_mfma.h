// Convolution with the exact quire (paper Sec. 2, Sec. 3.1, Sec. 3.3) on the integer matrix cores for posit(8,1), posit(8,2),
// posit(10,1), posit(12,1) and posit<16,1>: the implicit-GEMM form of conv_p8_mfma.h with the digit planes of dig_planes.h.
//
// Forward and backward-data: rows of the product are output channels, columns output positions (n, oh, ow), the reduction
// runs tap-major, channel-minor, so that 16 consecutive reduction indices are 16 channels of ONE input pixel.  One launch
// rewrites the gathered tensor as [pixel (n, h, w)][group of 16 channels][plane][16 bytes] and the weights in the row-block
// layout of the matrix product; the product kernel gathers: every lane of a copy names its own 16 bytes (the pixel its
// column reads for that tap, or a block of zeros), and the copy lands in LDS in lane order, which is the operand layout.
// Backward-data takes the weights transposed and flipped, NaR as zero (the outputs a NaR weight reaches are marked by the
// pass that follows, as for the other backward-data kernels).
//
// Backward-weight: rows are output channels, columns (c, r, s) and, for the bias gradient, one column of ones; the reduction
// runs position-major, image-minor, so that 16 consecutive indices are 16 images at one pixel, and x is gathered likewise.
// The reduction is cut into slices whose sums a merging launch adds and rounds.
//
// Which window of digits serves is decided on the device as for the matrix product: a kernel of four planes and one of
// eight are launched, the one decided on does the work.
#pragma once

#include "conv_b8.h"
#include "conv_desc.h"
#include "gemm_dig_mfma.h"

namespace pnn {

// Formats these kernels serve, and the planes of their wide kernel.
template <class F>
constexpr bool dig_conv_format() { return F::N <= 16 && F::ES != 0 && DigFormat<F>::COVER; }
template <class F>
constexpr int dig_conv_wide() { return DigFormat<F>::NP2 <= 4 ? 4 : 8; }

constexpr int DCM_MAXK16 = 512;  // most (tap, channel group) pairs, padding included

struct DigConvPlan {
    bool ok;
    int which;                 // 0 forward, 1 backward-data
    int NI, CI, HI, WI;        // the gathered tensor: x (forward) or dy (backward-data)
    int HO, WO, MO;            // output extents per image and output channels
    int R, S, offh, offw;      // tap (r, s) of output (oh, ow) reads input (oh sh + r - offh, ow sw + s - offw)
    int sh, sw;
    int WK, WC;                // the weight tensor is [WK][WC][R][S]
    int Cg, K16, KB;           // channel groups of 16, reduction length in 16s, k blocks of 32
    int WY, RBA;               // row blocks of 32 of a workgroup (DigConvShape), padded row blocks of the weights
    int64_t P;                 // output positions NI * HO * WO
    size_t w_bytes, act_bytes;
    // behind the planes: 256 bytes of zeros, 256 of decision, the scan's results
    size_t total() const { return w_bytes + act_bytes + 512 + DIG_STAT_BYTES; }
};

// posit(8,1) and posit(8,2) have the byte-gather kernel beside this one: whether these four launches pay, by an estimate fitted
// like b8_conv_us to layers whose operands four planes hold (off by 8 to 19 %).  Short reductions and one or two input channels
// under a large filter stay there: posit(8,1) backward-data of 64 images of 16 channels at 16 x 16 to 16, 1 x 1, 12.7 us there
// and 19.6 here; forward of 32 images of 1 channel at 32 x 32 to 32, 7 x 7, 20 and 36.  The factors are those that lost least
// over 2370 layers timed on both with blocks of 32 x 128 outputs: 15 of 1675 backward-data passes more than 6 % slower than here, 27 than there (estimates
// alike: 28 and 14; at 1.05 and 1.2: 78 and 8; posit(8,2), 24 images of 13 channels at 14 x 14 to 9, 5 x 5, 43 there and 26 here).  With the blocks of 16 x 32 per wave the line
// lies where it did: of 1685 layers of all three passes timed on both, 10 more than 3 % slower than on the other, a mean of 0.1 % lost.  Weights over
// most of the range of posit(8,2) take the wide kernel, at up to twice the time.
template <class F>
inline bool dig_conv_pays(const DigConvPlan& p) {
    const double groups = (double)(p.RBA / p.WY) * (double)((p.P + 32 * (4 / p.WY) - 1) / (32 * (4 / p.WY)));
    const double waves = groups > 256 ? groups / 256 - 1 : 0, mb = (double)p.NI * p.HI * p.WI * p.Cg * 16 / (1 << 20);
    const double here = F::ES == 1 ? 16.7 + 0.82 * p.KB * (1 + 0.5 * waves) + 2.2 * mb + 2.8 * waves : 19.1 + 0.77 * p.KB * (1 + 0.5 * waves) + 2.2 * mb + 2.6 * waves;
    return b8_conv_us<F>(false, (int)p.P, p.MO, p.CI * p.R * p.S) >= (p.which == 1 ? 0.95 : F::ES == 1 ? 1.0 : 1.1) * here;
}

template <class F>
inline DigConvPlan dig_conv_plan(int which, const ConvGeom& g) {
    DigConvPlan p;
    p.ok = false;
    p.which = which;
    if (!dig_conv_format<F>() || which > 1 || (which == 1 && (g.sh != 1 || g.sw != 1))) return p;
    p.NI = g.N; p.R = g.R; p.S = g.S; p.WK = g.K; p.WC = g.C; p.sh = g.sh; p.sw = g.sw;
    if (which == 0) {
        p.CI = g.C; p.HI = g.H; p.WI = g.W; p.HO = g.OH; p.WO = g.OW; p.MO = g.K; p.offh = g.ph; p.offw = g.pw;
    } else {
        p.CI = g.K; p.HI = g.OH; p.WI = g.OW; p.HO = g.H; p.WO = g.W; p.MO = g.C; p.offh = g.R - 1 - g.ph; p.offw = g.S - 1 - g.pw;
    }
    if (p.NI <= 0 || p.CI <= 0 || p.HI <= 0 || p.WI <= 0 || p.HO <= 0 || p.WO <= 0 || p.MO <= 0) return p;
    constexpr int slots = dig_conv_wide<F>();
    p.Cg = (p.CI + 15) / 16;
    p.P = (int64_t)p.NI * p.HO * p.WO;
    const int64_t pin = (int64_t)p.NI * p.HI * p.WI, k16 = (int64_t)g.R * g.S * p.Cg;
    if (k16 + 1 > DCM_MAXK16 || p.HI > 16384 || p.WI > 16384 || p.HO > 16384 || p.WO > 16384 || g.R > 4096 || g.S > 4096) return p;
    if (pin * p.Cg * slots >= ((int64_t)1 << 30) || p.P >= ((int64_t)1 << 30) || p.MO > 65536 || p.P * p.MO >= ((int64_t)1 << 40)) return p;
    if (!conv_gather_fits(p.NI, p.HI, p.WI, p.HO, p.WO, g.R, g.S, p.offh, p.offw, g.sh, g.sw, p.Cg * slots)) return p;
    p.K16 = (int)k16;
    p.KB = (p.K16 + 1) / 2;
    // Four launches: below these sizes the byte-gather kernel of the 8-bit formats is faster forward (15 M products: 25 against
    // 28 us; its backward-data takes 75), the generic kernel of the others is not (97 against 28 us).
    const int64_t least = F::N == 8 && which == 0 ? (int64_t)1 << 25 : (int64_t)1 << 22;
    if (p.P * p.MO * p.CI * g.R * g.S < least || p.P < 2048) return p;
    p.WY = p.MO > 32 ? 2 : 1;
    p.RBA = (int)((p.MO + 32 * p.WY - 1) / (32 * p.WY)) * p.WY;
    p.w_bytes = (size_t)p.KB * p.RBA * slots * 1024;
    p.act_bytes = (size_t)pin * p.Cg * slots * 16;
    if constexpr (F::N == 8) {
        if (p8_conv_eligible(which, g) && !dig_conv_pays<F>(p)) return p;
    }
    p.ok = true;
    return p;
}

// The digit word of a pattern: through a table in LDS for the 8-bit formats.
template <class F, int NP>
struct DigLookup {
    typedef typename DigWord<NP>::T W;
    const uint64_t* tab;
    int base;
    __device__ __forceinline__ W operator()(uint32_t p) const {
        if constexpr (F::N == 8) return (W)tab[p];
        else return dig_word<F, NP>(p & F::MASK, base);
    }
};

// 16 patterns a fixed step apart; beyond n: zeros.
template <class T>
__device__ __forceinline__ void dig_load16(const T* q, int64_t step, int n, uint32_t (&pat)[16]) {
#pragma unroll
    for (int b = 0; b < 16; ++b) pat[b] = b < n ? (uint32_t)q[b * step] : 0u;
}

// A wave's digits change hands in LDS before they are stored, so that a store instruction writes runs of the planes and not
// 16 bytes in every 64 (NP planes) or more (posit(8,2), 4 M elements and fewer: 9.4 to 8.4 us on average).  Slot of plane j
// of thread s: rows of NP slots, rotated so that sixteen threads reach sixteen different bank groups both ways.
template <int NP>
__device__ __forceinline__ int dig_xch(int s, int j) { return s * NP + (j ^ ((s >> (NP == 4 ? 2 : 1)) & (NP - 1))); }

// LDS accesses of a wave complete in order: only the compiler has to keep them so.
__device__ __forceinline__ void dig_wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <class F, int NP, int PX>
__device__ __forceinline__ void dig_conv_planes(const typename Storage<F::N>::T* __restrict__ src, int HW, int64_t pixels, uint4* __restrict__ act,
                                                const typename Storage<F::N>::T* __restrict__ w, const DigConvPlan& p, uint4* __restrict__ wdst,
                                                uint4* __restrict__ zero, unsigned wblocks, const DigInfo& d, uint64_t* tab, uint4* xch) {
    typedef typename Storage<F::N>::T T;
    typedef typename DigWord<NP>::T W;
    const int t = threadIdx.x;
    const bool weights = blockIdx.x < wblocks;
    const DigLookup<F, NP> word{tab, weights ? d.base[1] : d.base[0]};
    if constexpr (F::N == 8) {
        tab[t] = dig_word<F, NP>((uint32_t)t, word.base);
        __syncthreads();
    }
    if (weights) {
        const int64_t idx = (int64_t)blockIdx.x * 256 + t;
        if (idx < 16) zero[idx] = make_uint4(0, 0, 0, 0);  // what the product kernel reads for padding (no memset: graph capture)
        if (idx >= (int64_t)p.KB * p.RBA * 64) return;
        const int lane = (int)(idx & 63);
        const int rb = (int)((idx >> 6) % p.RBA), kb = (int)((idx >> 6) / p.RBA);
        const int row = rb * 32 + (lane & 31), k16 = kb * 2 + (lane >> 5);
        uint32_t pat[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) pat[b] = 0;
        if (row < p.MO && k16 < p.K16) {
            const int tap = k16 / p.Cg, cg = k16 - tap * p.Cg;
            const int r = tap / p.S, s = tap - r * p.S;
            const int nch = p.CI - cg * 16 < 16 ? p.CI - cg * 16 : 16;
            // forward: w[row][ch][r][s]; backward-data: w[ch][row][R-1-r][S-1-s]
            const int64_t rs = (int64_t)p.R * p.S;
            const T* q = p.which == 0 ? w + ((int64_t)row * p.WC + cg * 16) * rs + r * p.S + s
                                      : w + ((int64_t)cg * 16 * p.WC + row) * rs + (p.R - 1 - r) * p.S + (p.S - 1 - s);
            dig_load16<T>(q, p.which == 0 ? rs : rs * p.WC, nch, pat);
        }
        W wd[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) wd[b] = p.which != 0 && (pat[b] & F::MASK) == F::NAR ? (W)0 : word(pat[b]);
        uint32_t pl[NP][4];
        dig_planes_of<NP>(wd, pl);
        uint4* out = wdst + ((int64_t)(kb * p.RBA + rb) * NP) * 64 + lane;
#pragma unroll
        for (int i = 0; i < NP; ++i) out[i * 64] = make_uint4(pl[i][0], pl[i][1], pl[i][2], pl[i][3]);
        return;
    }
    // channel groups run fastest over the threads, so a wave's digits are runs of Cg * NP * 16 bytes, PX pixels apart
    const uint32_t total = (uint32_t)(pixels / PX) * (uint32_t)p.Cg;  // PX divides HW, hence pixels
    const uint32_t first = (blockIdx.x - wblocks) * 256u + ((uint32_t)t & ~63u), idx = first + ((uint32_t)t & 63u);
    uint32_t in[16];  // PX patterns of one channel
#pragma unroll
    for (int b = 0; b < 16; ++b) in[b] = 0;
    if (idx < total) {
        const uint32_t pg = idx / (uint32_t)p.Cg, cg = idx - pg * (uint32_t)p.Cg, pix = pg * PX;
        const uint32_t img = pix / (uint32_t)HW, hw = pix - img * (uint32_t)HW;
        const T* q = src + ((int64_t)img * p.CI + cg * 16) * (int64_t)HW + hw;
        const int nch = p.CI - (int)cg * 16 < 16 ? p.CI - (int)cg * 16 : 16;
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            if (b >= nch) continue;
            if (PX > 1) in[b] = *reinterpret_cast<const uint32_t*>(q + (int64_t)b * HW);
            else in[b] = q[(int64_t)b * HW];
        }
    }
    uint4* const mine = xch + (t >> 6) * (64 * NP);
#pragma unroll
    for (int px = 0; px < PX; ++px) {
        W wd[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) wd[b] = word((in[b] >> (8 * (int)sizeof(T) * px)) & (sizeof(T) == 1 ? 0xFFu : 0xFFFFu));
        uint32_t pl[NP][4];
        dig_planes_of<NP>(wd, pl);
#pragma unroll
        for (int i = 0; i < NP; ++i) mine[dig_xch<NP>(t & 63, i)] = make_uint4(pl[i][0], pl[i][1], pl[i][2], pl[i][3]);
        dig_wave_fence();
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const uint32_t s = (uint32_t)(i * 64 + (t & 63)) / NP, j = (uint32_t)(t & 63) % NP;  // plane j of thread s of the wave
            if (first + s < total) {
                const uint32_t pg = (first + s) / (uint32_t)p.Cg, cg = first + s - pg * (uint32_t)p.Cg;
                act[((int64_t)(pg * PX + px) * p.Cg + cg) * NP + j] = mine[dig_xch<NP>(s, j)];
            }
        }
        dig_wave_fence();
    }
}

// One launch rewrites both operands; the first wblocks workgroups take the weights (few threads, long chains of loads:
// started first), the rest the gathered tensor, one thread per channel group and PX consecutive pixels (as many as a 32-bit
// load holds, or one); consecutive threads take consecutive pixels.
template <class F, int PX>
__global__ __launch_bounds__(256) void dig_conv_digits_kernel(const typename Storage<F::N>::T* __restrict__ src, int HW, int64_t pixels, uint4* __restrict__ act,
                                                              const typename Storage<F::N>::T* __restrict__ w, DigConvPlan p, uint4* __restrict__ wdst,
                                                              uint4* __restrict__ zero, unsigned wblocks, const void* __restrict__ stats,
                                                              DigInfo* __restrict__ info) {
    typedef DigFormat<F> D;
    __shared__ uint64_t tab[F::N == 8 ? 256 : 1];
    const DigInfo d = dig_read_decision<F, false>(stats, info, D::NP1 == 4, blockIdx.x == 0);
    __shared__ uint4 xch[256 * dig_conv_wide<F>()];
    if (D::NP1 == 4 && d.np == 4) dig_conv_planes<F, 4, PX>(src, HW, pixels, act, w, p, wdst, zero, wblocks, d, tab, xch);
    else dig_conv_planes<F, dig_conv_wide<F>(), PX>(src, HW, pixels, act, w, p, wdst, zero, wblocks, d, tab, xch);
}

struct DigConvArgs {
    const uint4* Ad;      // weight planes
    const uint4* act;     // planes of the gathered tensor
    const uint4* zero;    // 256 bytes of zeros
    const DigInfo* info;
    int np;               // the decision this kernel serves
    int RBA, KB, K16, Cg;
    int HI, WI, HO, WO, S, offh, offw, sh, sw, MO, P;
    const void* bias;
    void* out;
    FmtRT fin, fout;
    int tiles_m;
    BwdDataNar nar;       // with weights only in the last launch of a backward-data call
};

// 128-bit quire from the sums' integer (units of minpos^2 2^at), for adding a bias: at < 0 drops zero bits, at >= 0 stays
// within 128 bits (see dig_add_bias).
template <int L>
__device__ __forceinline__ unsigned __int128 dig_to_quire(const uint32_t (&q)[L], int at) {
    const uint32_t top = L >= 4 ? q[L >= 4 ? 3 : 0] : (uint32_t)((int32_t)q[L - 1] >> 31);
    const unsigned __int128 x = ((unsigned __int128)(((uint64_t)top << 32) | q[2]) << 64) | (((uint64_t)q[1] << 32) | q[0]);
    return at >= 0 ? x << at : (unsigned __int128)((__int128)x >> -at);
}

// Rounds and stores rows first, first + STEP, ... of one column, two in flight; bias: 128-bit addends by row, in LDS.
template <int L, class T, int STEP, class Value, class IsNar>
__device__ __forceinline__ void dig_store_rows_bias(int first, int rows, const DigRound& d, T* dst, int64_t ld, const uint4* bias, const Value& value,
                                                    const IsNar& is_nar) {
    const int qfrac = 2 * d.fin.maxs();
#pragma unroll 1
    for (int lr0 = first; lr0 < rows; lr0 += 2 * STEP) {
        uint32_t res[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int lr = lr0 + u * STEP < rows ? lr0 + u * STEP : rows - 1;
            uint32_t q[L];
            value(lr, q);
            const uint4 b = bias[lr];
            const unsigned __int128 x = dig_to_quire<L>(q, d.at) + (((unsigned __int128)(((uint64_t)b.w << 32) | b.z) << 64) | (((uint64_t)b.y << 32) | b.x));
            const uint32_t s[4] = {(uint32_t)x, (uint32_t)(x >> 32), (uint32_t)(x >> 64), (uint32_t)(x >> 96)};
            const uint32_t v = dig_round_limbs<4, sizeof(T) == 4>(s, qfrac, d.fout);
            res[u] = is_nar(lr) ? d.fout.nar() : v;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (lr0 + u * STEP < rows) dst[(int64_t)(lr0 + u * STEP) * ld] = (T)res[u];
    }
}

// Four waves: 32 x 64 outputs (WY = 1: layers of at most 32 output channels) or 64 x 32 (rows: output channels, columns: positions).
template <int WY>
struct DigConvShape {
    static constexpr int NA = WY, NB = 2 / WY;  // row and column blocks of 32
    static constexpr int TR = 32 * NA, TC = 32 * NB;
};

// A wave owns 16 x 32 outputs, two blocks of v_mfma_i32_16x16x64_i8 whose 2 NP - 1 sums take 56 registers for four planes and 120 for
// eight, so that three or four and two workgroups share a CU (with blocks of 32 x 32 outputs two and one, and twice the outputs in a workgroup:
// a last round of workgroups twice as long).  A step takes a pair of k blocks of 32: a lane's 16 reduction indices come from block l / 32 of it.
// Room for one pair, whose operand quads (24 with eight planes) go to registers before the next pair's copies start; the other workgroups multiply meanwhile.  Or, four
// planes, a ring of two pairs, the next one copied while a pair is multiplied.
// Prologue and rounding weigh as much as the matrix instructions of a short reduction: four planes are all multiplied, and outputs of at most 16 bits
// are rounded through binary64 in registers and stored from there (the kernel alone with blocks of 32 x 32, 128 images of 32 channels at 32 x 32, posit(8,2), 3 x 3 to 32
// channels: 31 us, with integers of 96 bits through LDS 36).  Eight planes without NaR: only the planes that hold digits (with the same blocks, weights over most of the range
// of posit(8,2) 46 us, all 8 x 8 pairs 61; the call then and now, patterns at random for weights, 119 and 90).  us a call, 32 x 32 -> now: posit<16,1> backward-data of 100 images of 30 channels at 27 x 27 to 45, 3 x 3, 54.9 and 45.3; forward of 46 of 48 at
// 22 x 22 to 39, 5 x 5, stride 2, 49.0 and 32.0.  An odd last block (dig_single_mma; beside a block of
// zeros before): posit(12,1) backward-data of 10 of 48 at 43 x 43 to 24, 3 x 3, 25.0 and 23.6.
// ONE: four planes with one pair in LDS (30 KB, read and refilled as with eight planes) and a fourth workgroup on the CU, whose registers the bias, fetched behind the loop, leaves
// free.  us a call, 32 x 32 blocks, two pairs, one: posit(12,1) backward-data of 74 images of 4 channels at 51 x 51 to 21, 1 x 1, 43.7, 48.1, 43.5; 3490 passes of
// three k blocks and more 0.82 of the time of the 32 x 32 blocks in the mean, 0.85 with two pairs, 1 and 107 of them more than 3 % slower than with those (most where 768
// workgroups, three to a CU, leave a short second round); 1763 of one or two k blocks 0.94 and 1.00, 9 and 680.  Two pairs stay where one round of three holds the launch and the reduction is long enough for its copies to
// run ahead: up to 768 workgroups and more than 8 k blocks, 19 to 48 blocks 2 % and longer ones 4 % faster than with one pair.
template <int NP, int WY, bool ONE>
__device__ __forceinline__ void dig_conv_tile(const DigConvArgs& a, int tm, int tn) {
    typedef DigConvShape<WY> Sh;
    constexpr int NC = 2 * NP - 1, L = dig_limbs<NP>(), NA = Sh::NA, NB = Sh::NB, TR = Sh::TR, TC = Sh::TC, WAVES = 4, THREADS = 256;
    constexpr int PAIRS = NP <= 4 && !ONE ? 2 : 1;  // held in LDS
    constexpr int RPB = (NA + NB) * NP;           // runs of 1 KB per k block
    static_assert((NA * NP) % WAVES == 0 && (NB * NP) % WAVES == 0 && WAVES % NB == 0, "copies spread evenly over the waves");
    constexpr int ARUNS = NA * NP / WAVES;        // weight runs copied by a wave
    constexpr int GRUNS = NB * NP / WAVES;        // gathered runs: planes of one column block
    // one LDS object (see dig_gemm_kernel): the ring and the (tap, channel group) table; 52 KB, three workgroups to a CU, or 30 KB.  Behind the
    // loop the outputs' integers, the bias addends and the NaR flags take the ring.
    constexpr int VALS = L * TR * TC / 4, BEHIND = VALS + TR + (TR + TC) / 4;  // words of 16 bytes
    constexpr int PAIRW = 2 * PAIRS * RPB * 64, RING = PAIRW > BEHIND ? PAIRW : BEHIND, KTAB = DCM_MAXK16 / 2;
    __shared__ uint4 lds[RING + KTAB];
    uint4* const stage = lds;
    int2* const ktab = reinterpret_cast<int2*>(lds + RING);
    uint4* const badd = stage + VALS;
    uint32_t* const rowv = reinterpret_cast<uint32_t*>(badd + TR);
    uint32_t* const colv = rowv + TR;

    const int t = threadIdx.x;
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wr = w % (2 * NA), wc = w / (2 * NA);  // block of 16 rows, block of 32 columns
    const int pairs = (a.KB + 1) / 2;

    for (int k = t; k < 4 * pairs; k += THREADS) {
        int2 e = make_int2(0, 0x7FFF);  // beyond the reduction: a row offset no pixel has
        if (k < a.K16) {
            const int tap = k / a.Cg, cg = k - tap * a.Cg;
            const int r = tap / a.S, s = tap - r * a.S;
            const int dh = r - a.offh, dw = s - a.offw;
            e.x = ((dh * a.WI + dw) * a.Cg + cg) * NP;
            e.y = (int)(((uint32_t)dh & 0xFFFFu) | ((uint32_t)dw << 16));
        }
        ktab[k] = e;
    }

    // weights: wave w copies ARUNS of the k block's NA NP runs, wave-uniform addresses
    const uint4* const asrc = a.Ad + ((int64_t)tm * NA * NP + w * ARUNS) * 64 + lane;
    const int64_t a_kb = (int64_t)a.RBA * NP * 64;
    // gathered tensor: wave w takes GRUNS planes of column block w / (WAVES / NB); lane l of a copy serves column l % 32 of the
    // block and the 16 reduction indices of half l / 32
    constexpr int WPB = WAVES / NB;  // waves per column block
    const int cb = w / WPB, pl0 = (w % WPB) * GRUNS;
    const int hw_o = a.HO * a.WO;
    int oh = -40000, ow = 0, base = 0;  // beyond the positions: no tap brings this into the tensor
    {
        const int pos = tn * TC + cb * 32 + (lane & 31);
        if (pos < a.P) {
            const int img = pos / hw_o, rem = pos - img * hw_o;
            const int h = rem / a.WO;
            oh = h * a.sh;
            ow = (rem - h * a.WO) * a.sw;
            base = ((img * a.HI + oh) * a.WI + ow) * a.Cg * NP;
        }
    }
    const uint4* const actq = a.act + pl0;
    const uint4* const zeroq = a.zero;
    auto issue = [&](int p) {  // the two k blocks of pair p, or the last one
        const uint4* src[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int2 e = ktab[p * 4 + 2 * h + (lane >> 5)];
            // (Both halves in one read: left to itself the compiler reads the offset only where the row is inside, behind a wait of its
            // own; posit<16,1>, 77 images of 64 channels at 37 x 37, 3 x 3 to 20, forward 76.6 us and 74.5, 63 of 80 at 18 x 18, 5 x 5 to 55,
            // backward-data 101.9 and 95.5.)
            asm("" : "+v"(e.x), "+v"(e.y));
            const int dh = (int)(short)(e.y & 0xFFFF), dw = e.y >> 16;
            const int ih = oh + dh, iw = ow + dw;
            const bool inside = ((unsigned)ih < (unsigned)a.HI) & ((unsigned)iw < (unsigned)a.WI);
            src[h] = inside ? actq + (base + e.x) : zeroq;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kb = 2 * p + h;
            if (kb >= a.KB) break;
            uint4* buf = stage + (kb & (2 * PAIRS - 1)) * (RPB * 64);
            const uint4* as = asrc + (int64_t)kb * a_kb;
#pragma unroll
            for (int c = 0; c < ARUNS; ++c)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(as + c * 64),
                                                 (__attribute__((address_space(3))) void*)(buf + (w * ARUNS + c) * 64), 16, 0, 0);
#pragma unroll
            for (int c = 0; c < GRUNS; ++c)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[h] + c),
                                                 (__attribute__((address_space(3))) void*)(buf + (NA * NP + cb * NP + pl0 + c) * 64), 16, 0, 0);
        }
    };

    const int a_nar = __builtin_amdgcn_readfirstlane(a.info->nar[1]), b_nar = __builtin_amdgcn_readfirstlane(a.info->nar[0]);
    const int at = __builtin_amdgcn_readfirstlane(a.info->base[0] + a.info->base[1]);
    const bool by_f64 = NP <= 4 && a.fout.n <= 16;
    __syncthreads();  // ktab
    issue(0);
    uint32_t bias_nar = 0;
    uint4 bias_add = make_uint4(0, 0, 0, 0);
    auto load_bias = [&]() {
        if (!a.bias || t >= TR || tm * TR + t >= a.MO) return;
        const uint32_t bp = dig_load_pattern(a.bias, tm * TR + t, a.fin.n);
        bias_nar = bp == a.fin.nar() ? 1u : 0u;
        if (by_f64) {
            const double v = bias_nar ? 0.0 : dig_f64_of_pattern(bp, a.fin, 2 * a.fin.maxs() - at);
            bias_add = make_uint4(f64_lo(v), f64_hi(v), 0u, 0u);
        } else {
            const unsigned __int128 v = (unsigned __int128)dig_bias_value(bp, a.fin);
            bias_add = make_uint4((uint32_t)v, (uint32_t)(v >> 32), (uint32_t)(v >> 64), (uint32_t)(v >> 96));
        }
    };
    if (!ONE) load_bias();  // while the first blocks come in

    dig_v4i acc[2][NC];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < NC; ++s) acc[h][s] = dig_v4i{0, 0, 0, 0};
    uint32_t row_nar = 0, col_nar[2] = {0, 0};
    // lane l of a fragment: row or column l % 16 of its block, reduction indices 16 ((l / 16) % 2) .. of k block l / 32 of the pair
    const uint4* const lane0 = stage + (lane >> 5) * (RPB * 64) + ((lane >> 4) & 1) * 32 + (lane & 15);
    const uint4* const sa0 = lane0 + (wr >> 1) * NP * 64 + (wr & 1) * 16;
    const uint4* const sb0 = lane0 + (NA + wc) * NP * 64;
    auto loop = [&](auto ta, auto tb) {
        constexpr int TA = ta, TB = tb;
        for (int p = 0; p < a.KB / 2; ++p) {
            // This wave's copies of pair p have landed; behind the barrier everyone's have, and everyone's reads of the pair before have
            // been consumed, so its half of the ring takes the next.
            __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
            pcm_ring_barrier();
            if (PAIRS == 2 && p + 1 < pairs) issue(p + 1);
            const int half = (p & (PAIRS - 1)) * (2 * RPB * 64);
            DigPair<NP> f;
            f.template load<0, TA, TB>(sa0 + half, sb0 + half);
            if (PAIRS == 1 && p + 1 < pairs) {
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): read; behind the barrier everyone has
                pcm_ring_barrier();
                issue(p + 1);
            }
            if (TA == NP && TB == NP) dig_pair_markers<NP>(a_nar, b_nar, f, row_nar, col_nar);
            dig_pair_mma<NP, 0, TA, 0, TB>(f, acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if constexpr (NP <= 4) {
        loop(dig_int<NP>(), dig_int<NP>());
    } else {  // the planes that hold anything
        const int ua = __builtin_amdgcn_readfirstlane(a.info->used[1]), ub = __builtin_amdgcn_readfirstlane(a.info->used[0]);
        dig_for_planes<NP>(a_nar || b_nar ? NP : ua, ub, loop);
    }
    if (a.KB & 1) {
        __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
        pcm_ring_barrier();
        const int at = ((pairs - 1) & (PAIRS - 1)) * (2 * RPB * 64) - (lane >> 5) * (RPB * 64);
        dig_single_mma<NP>(sa0 + at, sb0 + at, lane, a_nar, b_nar, row_nar, col_nar, acc);
    }
    __syncthreads();  // the last pair is read: the ring is free
    if (ONE) load_bias();
    if (t < TR) {
        rowv[t] = bias_nar;
        badd[t] = bias_add;
    }
    if (a_nar) __syncthreads();  // the flags of the rows come on top

    uint32_t* const vals = reinterpret_cast<uint32_t*>(stage);
    row_nar = dig_pair_across(row_nar);
#pragma unroll
    for (int h = 0; h < 2; ++h) col_nar[h] = dig_pair_across(col_nar[h]);
    if (lane < 16) {
        if (wc == 0 && row_nar) rowv[wr * 16 + lane] = 1u;  // every wave of a row block saw the same rows
        if (wr == 0) {
#pragma unroll
            for (int h = 0; h < 2; ++h) colv[wc * 32 + 16 * h + lane] = col_nar[h];
        }
    }
    if constexpr (NP <= 4) {
        if (by_f64) {  // rounded and stored where the matrix instruction leaves them: four rows of one position per lane and block
            __syncthreads();
            const int rows = a.MO - tm * TR, lr0 = wr * 16 + 4 * (lane >> 4);
            const DigF64Round round(a.fout, 2 * a.fin.maxs() - at);
            const uint32_t nar = a.fout.nar();
            const uint4 fl = *reinterpret_cast<const uint4*>(rowv + lr0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int n = tn * TC + wc * 32 + 16 * h + (lane & 15);
                if (n >= a.P) continue;
                const int img = n / hw_o, rem = n - img * hw_o;
                const int64_t o = ((int64_t)img * a.MO + tm * TR) * hw_o + rem;
                const uint32_t flag[4] = {fl.x | col_nar[h], fl.y | col_nar[h], fl.z | col_nar[h], fl.w | col_nar[h]};
                double s[4], e[4];
                uint32_t v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    double hi, lo;
                    DigF64<NP>::parts(acc[h], u, hi, lo);
                    dig_two_sum(hi, lo, s[u], e[u]);
                }
                if (a.bias) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint2 b = *reinterpret_cast<const uint2*>(badd + lr0 + u);
                        dig_add_f64(s[u], e[u], f64_from_words(b.y, b.x));
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = flag[u] ? nar : round(s[u], e[u]);
                if (a.fout.n <= 8) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (lr0 + u < rows) ((uint8_t*)a.out)[o + (int64_t)(lr0 + u) * hw_o] = (uint8_t)v[u];
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (lr0 + u < rows) ((uint16_t*)a.out)[o + (int64_t)(lr0 + u) * hw_o] = (uint16_t)v[u];
                }
            }
            return;
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int lr = wr * 16 + 4 * (lane >> 4) + r;
            uint32_t q[L];
            dig_combine<NP>(acc[h], r, q);
#pragma unroll
            for (int l = 0; l < L; ++l) vals[l * (TR * TC) + lr * TC + wc * 32 + 16 * h + (lane & 15)] = q[l];
        }
    __syncthreads();
    // neighbouring threads: neighbouring positions, every STEP-th row
    constexpr int STEP = THREADS / TC;
    const int col = t % TC, first = t / TC;
    const int n = tn * TC + col;
    if (n >= a.P) return;
    const int rows = a.MO - tm * TR < TR ? a.MO - tm * TR : TR;
    const uint32_t cnar = colv[col];
    const int img = n / hw_o, rem = n - img * hw_o;
    const int64_t o = ((int64_t)img * a.MO + tm * TR) * hw_o + rem;
    DigRound rd;
    rd.fin = a.fin;
    rd.fout = a.fout;
    rd.at = at;
    auto value = [&](int lr, uint32_t (&q)[L]) {
        lr = lr < TR ? lr : TR - 1;  // asked for beyond the rows, not stored
#pragma unroll
        for (int l = 0; l < L; ++l) q[l] = vals[l * (TR * TC) + lr * TC + col];
    };
    auto is_nar = [&](int lr) { return (cnar | rowv[lr < TR ? lr : TR - 1]) != 0; };
    if (a.bias) {
        if (rd.fout.n <= 8) dig_store_rows_bias<L, uint8_t, STEP>(first, rows, rd, (uint8_t*)a.out + o, hw_o, badd, value, is_nar);
        else if (rd.fout.n <= 16) dig_store_rows_bias<L, uint16_t, STEP>(first, rows, rd, (uint16_t*)a.out + o, hw_o, badd, value, is_nar);
        else dig_store_rows_bias<L, uint32_t, STEP>(first, rows, rd, (uint32_t*)a.out + o, hw_o, badd, value, is_nar);
    } else {
        if (rd.fout.n <= 8) dig_store_rows<L, uint8_t, STEP>(first, rows, rd, (uint8_t*)a.out + o, hw_o, value, is_nar);
        else if (rd.fout.n <= 16) dig_store_rows<L, uint16_t, STEP>(first, rows, rd, (uint16_t*)a.out + o, hw_o, value, is_nar);
        else dig_store_rows<L, uint32_t, STEP>(first, rows, rd, (uint32_t*)a.out + o, hw_o, value, is_nar);
    }
}

// The last launch of a backward-data call also marks what NaR weights reach, tile by tile: behind its own work, or, if another
// launch did that, right away (100 images of 30 channels at 27 x 27 to 45, posit<16,1>: 57.6 us with a launch of its own, 56.6 so;
// the posit<8,0> kernel, which has no spare launch, lost 1 to 4 % on large layers by it).
template <int NP, int WY, bool ONE>
__global__ __launch_bounds__(256, (NP > 4 ? 2 : ONE ? 4 : 3)) void dig_conv_kernel(DigConvArgs a) {
    typedef DigConvShape<WY> Sh;
    const bool mark = a.nar.w && __builtin_amdgcn_readfirstlane(a.info->nar[1]);
    // a position's row tiles and the positions that share its taps on one XCD; nothing is shared by a single row of 1 x 1 tiles
    const int tiles = a.tiles_m * ((a.P + Sh::TC - 1) / Sh::TC), id = dig_tile_id();
    if (id >= tiles) return;
    const int tile = a.tiles_m > 1 || a.K16 > a.Cg ? dig_xcd_order(id, tiles) : id, tm = tile % a.tiles_m, tn = tile / a.tiles_m;
    if (__builtin_amdgcn_readfirstlane(a.info->np) == a.np) dig_conv_tile<NP, WY, ONE>(a, tm, tn);
    if (mark) bwd_data_nar_tile<Sh::TR, Sh::TC>(a.nar, a.out, tm * Sh::TR, tn * Sh::TC);
}

template <int WY>
inline dim3 dig_conv_grid(int tiles_m, int64_t P) { return dig_tile_grid(tiles_m * ((P + DigConvShape<WY>::TC - 1) / DigConvShape<WY>::TC)); }

template <int NP, int WY>
inline hipError_t launch_dig_conv_shape(hipStream_t stream, const DigConvArgs& a) {
    const dim3 grid = dig_conv_grid<WY>(a.tiles_m, a.P);
    if (NP <= 4 && (a.KB <= 8 || (int64_t)grid.x * grid.z > 768)) hipLaunchKernelGGL((dig_conv_kernel<NP, WY, NP <= 4>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((dig_conv_kernel<NP, WY, false>), grid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int NP>
inline hipError_t launch_dig_conv_product(hipStream_t stream, const DigConvArgs& a, int WY) {
    return WY == 1 ? launch_dig_conv_shape<NP, 1>(stream, a) : launch_dig_conv_shape<NP, 2>(stream, a);
}

// in: x (forward) or dy (backward-data); workspace: [weight planes][planes of in][256 zeros][decision][scan]
template <class F>
inline hipError_t launch_dig_conv(hipStream_t stream, const DigConvPlan& p, const void* in, const void* w, const void* bias, void* out, int fout,
                                  void* workspace, const BwdDataNar& nar = BwdDataNar{}) {
    typedef typename Storage<F::N>::T T;
    typedef DigFormat<F> D;
    uint8_t* base = (uint8_t*)workspace;
    uint4* Ad = (uint4*)base;
    uint4* act = (uint4*)(base + p.w_bytes);
    uint4* zero = (uint4*)(base + p.w_bytes + p.act_bytes);
    DigInfo* info = (DigInfo*)(zero + 16);
    void* stats = (void*)(zero + 32);
    const int64_t pixels = (int64_t)p.NI * p.HI * p.WI;
    const int HW = p.HI * p.WI;
    const int64_t nx = pixels * p.CI, nw = (int64_t)p.WK * p.WC * p.R * p.S;
    const DigStatJob sx{in, 1, nx, nx, 0}, sw{w, 1, nw, nw, 0};
    hipLaunchKernelGGL((dig_stat_kernel<F, false>), dim3((unsigned)dig_stat_wgs<false>(), 2), dim3(1024), 0, stream, sx, sw, stats);
    PNN_CHECK_LAUNCH();
    const unsigned wblocks = (unsigned)(((int64_t)p.KB * p.RBA * 64 + 255) / 256);
    constexpr int PX = 4 / (int)sizeof(T);
    if (HW % PX == 0 && ((uintptr_t)in & 3u) == 0) {
        const unsigned ablocks = (unsigned)((pixels / PX * p.Cg + 255) / 256);
        hipLaunchKernelGGL((dig_conv_digits_kernel<F, PX>), dim3(wblocks + ablocks), dim3(256), 0, stream, (const T*)in, HW, pixels, act, (const T*)w, p, Ad,
                           zero, wblocks, stats, info);
    } else {
        const unsigned ablocks = (unsigned)((pixels * p.Cg + 255) / 256);
        hipLaunchKernelGGL((dig_conv_digits_kernel<F, 1>), dim3(wblocks + ablocks), dim3(256), 0, stream, (const T*)in, HW, pixels, act, (const T*)w, p, Ad,
                           zero, wblocks, stats, info);
    }
    PNN_CHECK_LAUNCH();
    DigConvArgs a;
    a.Ad = Ad; a.act = act; a.zero = zero; a.info = info;
    a.RBA = p.RBA; a.KB = p.KB; a.K16 = p.K16; a.Cg = p.Cg;
    a.HI = p.HI; a.WI = p.WI; a.HO = p.HO; a.WO = p.WO; a.S = p.S; a.offh = p.offh; a.offw = p.offw; a.sh = p.sh; a.sw = p.sw; a.MO = p.MO;
    a.P = (int)p.P;
    a.bias = bias; a.out = out;
    a.fin = fmt_of_code(code_of<F>());
    a.fout = fmt_of_code(fout);
    a.tiles_m = p.RBA / p.WY;
    a.nar = BwdDataNar{};
    if constexpr (D::NP1 == 4) {
        a.np = 4;
        const hipError_t e = launch_dig_conv_product<4>(stream, a, p.WY);
        if (e != hipSuccess) return e;
    }
    a.np = D::NP2;
    a.nar = nar;
    return launch_dig_conv_product<dig_conv_wide<F>()>(stream, a, p.WY);
}

// ---- backward-weight: dw[k][c][r][s] = sum over (n, oh, ow) of dy[n][k][oh][ow] x[n][c][oh sh + r - ph][ow sw + s - pw] ----

struct DigConvBwPlan {
    bool ok;
    ConvGeom g;
    int M, N, crs;             // outputs: K x CRS, or K x (CRS + 1) with the bias gradient as the last column
    int NG;                    // groups of 16 images
    int K16;                   // reduction length in 16s: OH OW NG
    int WY, RBA, KB;           // row blocks of 32 of a workgroup (DigConvShape), row blocks of dy's planes, k blocks (= splits * kb_per_split)
    int tiles_m, tiles_n;      // column tiles twice as wide as a workgroup's
    int splits, kb_per_split;
    size_t a_bytes, x_bytes, ones_bytes, part_bytes;
    // behind the planes and the blocks of ones: 256 bytes of zeros, 256 of decision, the scan's results, the partial sums
    size_t part_off() const { return a_bytes + x_bytes + ones_bytes + 512 + DIG_STAT_BYTES; }
    size_t total() const { return part_off() + part_bytes; }
};

// The same for the weight gradient, two launches and a merge: what is left to the byte-gather kernel are batches of one to three
// images (padded to 16 here; posit(8,1), one image of 64 channels at 64 x 64 to 64, 3 x 3: 43 us there, 87 here) and much
// input for few products.  Without a bias gradient the other path has a launch less.
template <class F>
inline bool dig_conv_bw_pays(const DigConvBwPlan& p, bool with_bias) {
    const ConvGeom& g = p.g;
    const double rows = (double)p.tiles_m * 32 * p.WY, cols = (double)p.tiles_n * 32 * (4 / p.WY), k = 16.0 * g.OH * g.OW * p.NG;
    const double mb = ((double)g.C * g.H * g.W * p.NG * 16 + k * rows) / (1 << 20), more = mb > 24 ? mb - 24 : 0;
    const double here = (F::ES == 1 ? 28.2 + 0.74 * mb : 30.5 + 1.14 * mb) + 1.1 * more + 1.88e-8 * k * rows * cols;
    return b8_conv_us<F>(true, p.crs, g.K, g.N * g.OH * g.OW) - (with_bias ? 0.0 : 8.0) >= 1.15 * here;
}

template <class F>
inline DigConvBwPlan dig_conv_bw_plan(const ConvGeom& g, bool with_bias) {
    DigConvBwPlan p;
    p.ok = false;
    p.g = g;
    if (!dig_conv_format<F>() || g.N <= 0 || g.C <= 0 || g.K <= 0) return p;
    constexpr int slots = dig_conv_wide<F>(), L = dig_limbs<slots>();
    const int64_t crs = (int64_t)g.C * g.R * g.S, P = (int64_t)g.N * g.OH * g.OW;
    if (crs > 65536 || g.K > 65536 || P < 2048 || P >= ((int64_t)1 << 28) || g.K * crs * P < ((int64_t)1 << 22)) return p;
    p.NG = (g.N + 15) / 16;
    const int64_t k16 = (int64_t)g.OH * g.OW * p.NG;
    if ((int64_t)g.C * g.H * g.W * p.NG * slots >= ((int64_t)1 << 30) || k16 >= ((int64_t)1 << 26) || g.H > 16384 || g.W > 16384) return p;
    p.K16 = (int)k16;
    p.M = g.K;
    p.crs = (int)crs;
    p.N = (int)crs + (with_bias ? 1 : 0);
    p.WY = p.M > 32 ? 2 : 1;
    const int tr = 32 * p.WY, tc = 32 * (4 / p.WY);
    p.tiles_m = (p.M + tr - 1) / tr;
    p.tiles_n = (p.N + tc - 1) / tc;
    p.RBA = p.tiles_m * p.WY;
    const int64_t kb_total = (k16 + 1) / 2, tiles = (int64_t)p.tiles_m * p.tiles_n;
    int64_t splits = (512 + tiles - 1) / tiles;                    // 512 pairs of workgroups: four to a compute unit
    if (splits > kb_total / 8) splits = kb_total / 8;              // at least 8 k blocks per slice
    if (splits < (kb_total + 510) / 511) splits = (kb_total + 510) / 511;  // and at most what int32 sums hold
    if (splits < 1) splits = 1;
    const int64_t kbps = (kb_total + splits - 1) / splits;
    splits = (kb_total + kbps - 1) / kbps;
    if (splits > 65535) return p;
    p.splits = (int)splits;
    p.kb_per_split = (int)kbps;
    p.KB = (int)(splits * kbps);
    p.a_bytes = (size_t)p.KB * p.RBA * slots * 1024;
    p.x_bytes = (size_t)g.C * g.H * g.W * p.NG * slots * 16;
    p.ones_bytes = (size_t)p.NG * slots * 16;
    if (p.a_bytes >= ((size_t)1 << 34)) return p;
    p.part_bytes = ((size_t)p.splits * p.M * p.N * L + (size_t)p.splits * (p.M + p.N)) * 4;
    if constexpr (F::N == 8) {
        if (p8_conv_eligible(2, g) && !dig_conv_bw_pays<F>(p, with_bias)) return p;
    }
    p.ok = true;
    return p;
}

// ablocks workgroups rewrite dy, the rest x (and the blocks of ones and zeros).
//   dy: workgroup (row block rb, image group g, chunk of positions) keeps the patterns of 16 images x 32 rows x POS positions
//       in LDS (read along the positions) and writes, per position and row, the planes of the 16 images.  Positions beyond
//       OH OW (up to the padded reduction length 2 KB) are written as zeros.
//   x:  one thread per (channel, PX consecutive pixels, image group); 16 loads a pixel-plane apart, coalesced along the pixels.
template <class F, int NP, int PX, int POS>
__device__ __forceinline__ void dig_conv_bw_planes(const typename Storage<F::N>::T* __restrict__ dy, const typename Storage<F::N>::T* __restrict__ x,
                                                   const DigConvBwPlan& p, uint4* __restrict__ Ad, uint4* __restrict__ xb, uint4* __restrict__ ones,
                                                   uint4* __restrict__ zero, unsigned ablocks, int chunks, const DigInfo& d, uint64_t* tab,
                                                   typename Storage<F::N>::T (*tile)[32][POS + 4 / (int)sizeof(typename Storage<F::N>::T)]) {
    typedef typename Storage<F::N>::T T;
    typedef typename DigWord<NP>::T W;
    constexpr int PW = 4 / (int)sizeof(T);  // positions per 32-bit word
    const int t = threadIdx.x;
    const bool rows = blockIdx.x < ablocks;
    const DigLookup<F, NP> word{tab, rows ? d.base[1] : d.base[0]};
    if constexpr (F::N == 8) tab[t] = dig_word<F, NP>((uint32_t)t, word.base);
    const ConvGeom& g = p.g;
    const int ohw = g.OH * g.OW;
    if (rows) {
        const int chunk = (int)(blockIdx.x % (unsigned)chunks);
        const int gi = (int)((blockIdx.x / (unsigned)chunks) % (unsigned)p.NG);
        const int rb = (int)(blockIdx.x / (unsigned)(chunks * p.NG));
        // loads in batches of eight before their LDS stores, so that eight are in flight per thread
        if (ohw % PW == 0 && ((uintptr_t)dy & 3u) == 0) {
            constexpr int WPR = POS / PW, ITEMS = 16 * 32 * WPR;  // 32-bit words per row, in all
#pragma unroll 1
            for (int base = 0; base < ITEMS; base += 8 * 256) {
                uint32_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int item = base + u * 256 + t, pair = item / WPR, q = item % WPR;
                    const int img = gi * 16 + (pair >> 5), row = rb * 32 + (pair & 31), pos = chunk * POS + q * PW;
                    v[u] = (img < g.N && row < g.K && pos < ohw) ? *reinterpret_cast<const uint32_t*>(dy + ((int64_t)img * g.K + row) * ohw + pos) : 0u;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int item = base + u * 256 + t, pair = item / WPR, q = item % WPR;
                    *reinterpret_cast<uint32_t*>(&tile[pair >> 5][pair & 31][q * PW]) = v[u];
                }
            }
        } else {
            constexpr int ITEMS = 16 * 32 * POS;
#pragma unroll 1
            for (int base = 0; base < ITEMS; base += 8 * 256) {
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int item = base + u * 256 + t, pair = item / POS, q = item % POS;
                    const int img = gi * 16 + (pair >> 5), row = rb * 32 + (pair & 31), pos = chunk * POS + q;
                    v[u] = (img < g.N && row < g.K && pos < ohw) ? dy[((int64_t)img * g.K + row) * ohw + pos] : (T)0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int item = base + u * 256 + t, pair = item / POS, q = item % POS;
                    tile[pair >> 5][pair & 31][q] = v[u];
                }
            }
        }
        __syncthreads();
        for (int item = t; item < POS * 32; item += 256) {
            const int pl = item >> 5, rr = item & 31;
            const int64_t k16 = (int64_t)(chunk * POS + pl) * p.NG + gi;
            if (k16 >= 2 * (int64_t)p.KB) continue;
            W wd[16];
#pragma unroll
            for (int b = 0; b < 16; ++b) wd[b] = word(tile[b][rr][pl]);
            uint32_t dg[NP][4];
            dig_planes_of<NP>(wd, dg);
            const int kb = (int)(k16 >> 1), lane = (int)(k16 & 1) * 32 + rr;
            uint4* out = Ad + ((int64_t)kb * p.RBA + rb) * (NP * 64) + lane;
#pragma unroll
            for (int i = 0; i < NP; ++i) out[i * 64] = make_uint4(dg[i][0], dg[i][1], dg[i][2], dg[i][3]);
        }
        return;
    }
    __syncthreads();  // the table
    const int64_t idx = (int64_t)(blockIdx.x - ablocks) * 256 + t;
    if (idx < 16) zero[idx] = make_uint4(0, 0, 0, 0);  // what the product kernel reads for padding (no memset: graph capture)
    if (idx < p.NG) {  // the column of ones, for the images the group really has
        W wd[16];
        const W one = word(F::NAR >> 1);
#pragma unroll
        for (int b = 0; b < 16; ++b) wd[b] = (int)idx * 16 + b < g.N ? one : (W)0;
        uint32_t dg[NP][4];
        dig_planes_of<NP>(wd, dg);
#pragma unroll
        for (int i = 0; i < NP; ++i) ones[idx * NP + i] = make_uint4(dg[i][0], dg[i][1], dg[i][2], dg[i][3]);
    }
    // as in dig_conv_planes: image groups run fastest over the threads, and a wave's digits change hands before the store
    // (whole calls, posit(8,2): 128 x 32 x 32 x 32 to 32 channels 76 to 72 us, 256 x 64 x 28 x 28 to 64 228 to 223)
    const int64_t planes = (int64_t)g.C * g.H * g.W;  // pixels of all channels of one image
    const uint32_t NG = (uint32_t)p.NG, total = (uint32_t)(planes / PX) * NG;
    const uint32_t first = (blockIdx.x - ablocks) * 256u + ((uint32_t)t & ~63u);
    uint32_t in[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) in[b] = 0;
    if (idx < total) {
        const uint32_t pg = (uint32_t)idx / NG, gi = (uint32_t)idx - pg * NG;
        const int nimg = g.N - (int)gi * 16 < 16 ? g.N - (int)gi * 16 : 16;
        const T* q = x + (int64_t)gi * 16 * planes + (int64_t)pg * PX;  // (c, h, w) as one index
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            if (b >= nimg) continue;
            if (PX > 1) in[b] = *reinterpret_cast<const uint32_t*>(q + (int64_t)b * planes);
            else in[b] = q[(int64_t)b * planes];
        }
    }
    static_assert(sizeof(T) * 16 * 32 * (POS + 4 / sizeof(T)) >= 256 * NP * 16, "the rows' tile has room for the exchange");
    uint4* const mine = reinterpret_cast<uint4*>(&tile[0][0][0]) + (t >> 6) * (64 * NP);
#pragma unroll
    for (int px = 0; px < PX; ++px) {
        W wd[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) wd[b] = word((in[b] >> (8 * (int)sizeof(T) * px)) & (sizeof(T) == 1 ? 0xFFu : 0xFFFFu));
        uint32_t dg[NP][4];
        dig_planes_of<NP>(wd, dg);
#pragma unroll
        for (int i = 0; i < NP; ++i) mine[dig_xch<NP>(t & 63, i)] = make_uint4(dg[i][0], dg[i][1], dg[i][2], dg[i][3]);
        dig_wave_fence();
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const uint32_t s = (uint32_t)(i * 64 + (t & 63)) / NP, j = (uint32_t)(t & 63) % NP;  // plane j of thread s of the wave
            if (first + s < total) {
                const uint32_t pg = (first + s) / NG, gi = first + s - pg * NG;
                xb[((int64_t)(pg * PX + px) * NG + gi) * NP + j] = mine[dig_xch<NP>(s, j)];
            }
        }
        dig_wave_fence();
    }
}

template <class F>
constexpr int dig_bw_positions() { return F::N == 8 ? 64 : 32; }

template <class F, int PX>
__global__ __launch_bounds__(256) void dig_conv_bw_digits_kernel(const typename Storage<F::N>::T* __restrict__ dy, const typename Storage<F::N>::T* __restrict__ x,
                                                                 DigConvBwPlan p, uint4* __restrict__ Ad, uint4* __restrict__ xb, uint4* __restrict__ ones,
                                                                 uint4* __restrict__ zero, unsigned ablocks, int chunks, const void* __restrict__ stats,
                                                                 DigInfo* __restrict__ info) {
    typedef DigFormat<F> D;
    typedef typename Storage<F::N>::T T;
    constexpr int POS = dig_bw_positions<F>();
    __shared__ uint64_t tab[F::N == 8 ? 256 : 1];
    __shared__ __attribute__((aligned(16))) T tile[16][32][POS + 4 / (int)sizeof(T)];
    const DigInfo d = dig_read_decision<F, false>(stats, info, D::NP1 == 4, blockIdx.x == 0);
    if (D::NP1 == 4 && d.np == 4) dig_conv_bw_planes<F, 4, PX, POS>(dy, x, p, Ad, xb, ones, zero, ablocks, chunks, d, tab, tile);
    else dig_conv_bw_planes<F, dig_conv_wide<F>(), PX, POS>(dy, x, p, Ad, xb, ones, zero, ablocks, chunks, d, tab, tile);
}

struct DigConvBwArgs {
    const uint4* Ad;      // dy's planes
    const uint4* xb;      // x's planes, image-minor
    const uint4* ones;    // per image group: the digits of 1 for the images it has
    const uint4* zero;    // 256 bytes of zeros
    const DigInfo* info;
    int np, RBA, kb_per_split;
    int NG, OH, OW, H, W, R, S, ph, pw, sh, sw;
    int crs, M, N;
    uint32_t* part;       // [slice][limb][M N]
    uint32_t* rowflag;    // [slice][M]
    uint32_t* colflag;    // [slice][N]
    int tiles_m;
    int splits;
    void* dw;
    void* dbias;
    FmtRT fin, fout;
    int qbits;
};

// Blocks, fragments and the step of two k blocks as in dig_conv_tile, one pair of them in LDS; workgroup (tile, z) reduces slice z and leaves
// one integer per output.  us a call, 32 x 32 -> now: posit(8,2),
// 128 images of 64 channels at 16 x 16 to 64, 3 x 3, 58.2 and 46.3; posit<16,1>, 48 of 58 at 48 x 48 to 7, 5 x 5, 147 and 112.
template <int NP, int WY>
__global__ __launch_bounds__(256, (NP <= 4 ? 4 : 2)) void dig_conv_bw_kernel(DigConvBwArgs a) {
    if (__builtin_amdgcn_readfirstlane(a.info->np) != a.np) return;
    typedef DigConvShape<WY> Sh;
    constexpr int NC = 2 * NP - 1, L = dig_limbs<NP>(), NA = Sh::NA, NB = Sh::NB, TR = Sh::TR, TC = Sh::TC;
    constexpr int RPB = (NA + NB) * NP;
    static_assert((NA * NP) % 4 == 0 && (NB * NP) % 4 == 0, "copies spread evenly over the waves");
    constexpr int ARUNS = NA * NP / 4, GRUNS = NB * NP / 4;
    __shared__ uint4 lds[2 * RPB * 64];
    uint4* const stage = lds;

    const int t = threadIdx.x;
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wr = w % (2 * NA), wc = w / (2 * NA);  // block of 16 rows, block of 32 columns
    // the tiles of a slice next to each other: they share its blocks
    const int id = dig_xcd_order((int)(blockIdx.x + blockIdx.y * gridDim.x), (int)(gridDim.x * gridDim.y));
    const int z = id / (int)gridDim.x, tile = id - z * (int)gridDim.x, tm = tile % a.tiles_m, tn = tile / a.tiles_m;
    const int kb0 = z * a.kb_per_split, nkb = a.kb_per_split;

    const int64_t a_kb = (int64_t)a.RBA * NP * 64;
    const uint4* asrc = a.Ad + kb0 * a_kb + ((int64_t)tm * NA * NP + w * ARUNS) * 64 + lane;
    // x: wave w gathers GRUNS planes of column block w / (4 / NB); lane l serves column l % 32 of the block and the 16
    // reduction indices (one pixel, one image group) of half l / 32
    constexpr int WPB = 4 / NB;
    const int cb = w / WPB, pl0 = (w % WPB) * GRUNS;
    const int n = tn * TC + cb * 32 + (lane & 31);
    int kind = 2, cbase = 0, dr = 0, ds = 0;  // kind 0: a column (c, r, s); 1: the column of ones; 2: beyond the columns
    if (n < a.crs) {
        const int rs = a.R * a.S;
        const int c = n / rs, tp = n - c * rs;
        const int r = tp / a.S, s = tp - r * a.S;
        kind = 0;
        cbase = c * a.H * a.W * a.NG * NP + pl0;
        dr = r - a.ph;
        ds = s - a.pw;
    } else if (n < a.N) {
        kind = 1;
    }
    // the reduction index of this lane's half, as (oh, ow, image group), stepped from k block to k block
    int oh, ow, gi;
    {
        const int k16 = kb0 * 2 + (lane >> 5);
        const int pos = k16 / a.NG;
        gi = k16 - pos * a.NG;
        oh = pos / a.OW;
        ow = pos - oh * a.OW;
    }
    auto issue = [&](int p) {  // the two k blocks of pair p, or the slice's last one
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (2 * p + h >= nkb) break;
            uint4* buf = stage + h * (RPB * 64);
            const uint4* as = asrc + (int64_t)(2 * p + h) * a_kb;
#pragma unroll
            for (int c = 0; c < ARUNS; ++c)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(as + c * 64),
                                                 (__attribute__((address_space(3))) void*)(buf + (w * ARUNS + c) * 64), 16, 0, 0);
            const uint4* s = a.zero;
            if (oh < a.OH) {  // inside the reduction (its padded end reads zeros)
                if (kind == 0) {
                    const int ih = oh * a.sh + dr, iw = ow * a.sw + ds;
                    if ((unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W) s = a.xb + (cbase + ((ih * a.W + iw) * a.NG + gi) * NP);
                } else if (kind == 1) {
                    s = a.ones + (gi * NP + pl0);
                }
            }
#pragma unroll
            for (int c = 0; c < GRUNS; ++c)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(s + c),
                                                 (__attribute__((address_space(3))) void*)(buf + (NA * NP + cb * NP + pl0 + c) * 64), 16, 0, 0);
            gi += 2;  // the next k block: two reduction indices of 16 further
            while (gi >= a.NG) {
                gi -= a.NG;
                if (++ow == a.OW) {
                    ow = 0;
                    ++oh;
                }
            }
        }
    };
    const int a_nar = __builtin_amdgcn_readfirstlane(a.info->nar[1]), b_nar = __builtin_amdgcn_readfirstlane(a.info->nar[0]);
    issue(0);
    dig_v4i acc[2][NC];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < NC; ++s) acc[h][s] = dig_v4i{0, 0, 0, 0};
    uint32_t row_nar = 0, col_nar[2] = {0, 0};
    const uint4* const lane0 = stage + (lane >> 5) * (RPB * 64) + ((lane >> 4) & 1) * 32 + (lane & 15);
    const uint4* const sa0 = lane0 + (wr >> 1) * NP * 64 + (wr & 1) * 16;
    const uint4* const sb0 = lane0 + (NA + wc) * NP * 64;
    const int pairs = (nkb + 1) / 2;
    auto loop = [&](auto ta, auto tb) {
        constexpr int TA = ta, TB = tb;
        for (int p = 0; p < nkb / 2; ++p) {
            __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));  // see dig_conv_tile
            pcm_ring_barrier();
            DigPair<NP> f;
            f.template load<0, TA, TB>(sa0, sb0);
            if (p + 1 < pairs) {
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
                pcm_ring_barrier();
                issue(p + 1);
            }
            if (TA == NP && TB == NP) dig_pair_markers<NP>(a_nar, b_nar, f, row_nar, col_nar);
            dig_pair_mma<NP, 0, TA, 0, TB>(f, acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if constexpr (NP <= 4) {
        loop(dig_int<NP>(), dig_int<NP>());
    } else {  // the planes that hold anything
        const int ua = __builtin_amdgcn_readfirstlane(a.info->used[1]), ub = __builtin_amdgcn_readfirstlane(a.info->used[0]);
        dig_for_planes<NP>(a_nar || b_nar ? NP : ua, ub, loop);
    }
    if (nkb & 1) {
        __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
        pcm_ring_barrier();
        const int at = -(lane >> 5) * (RPB * 64);
        dig_single_mma<NP>(sa0 + at, sb0 + at, lane, a_nar, b_nar, row_nar, col_nar, acc);
    }

    // ---- this slice's integers and NaR flags ----
    row_nar = dig_pair_across(row_nar);
#pragma unroll
    for (int h = 0; h < 2; ++h) col_nar[h] = dig_pair_across(col_nar[h]);
    const int64_t MN = (int64_t)a.M * a.N;
    const int n0 = tn * TC + wc * 32 + (lane & 15), m0 = tm * TR + wr * 16;
    // the first tile column stores the row flags of its tile row (the same in every column), the first tile row the column
    // flags: every entry is written, so the workspace needs no clearing
    if (lane < 16) {
        if (tn == 0 && wc == 0 && m0 + lane < a.M) a.rowflag[(int64_t)z * a.M + m0 + lane] = row_nar;
        if (tm == 0 && wr == 0) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (n0 + 16 * h < a.N) a.colflag[(int64_t)z * a.N + n0 + 16 * h] = col_nar[h];
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int nn = n0 + 16 * h;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + 4 * (lane >> 4) + r;
            uint32_t q[L];
            dig_combine<NP>(acc[h], r, q);
            if (m < a.M && nn < a.N) {
#pragma unroll
                for (int l = 0; l < L; ++l) a.part[((int64_t)z * L + l) * MN + (int64_t)m * a.N + nn] = q[l];
            }
        }
    }
}

// Adds the slices (eight threads per output take every eighth), wraps to the quire's width (a long reduction can leave it),
// rounds once, and routes the column of ones to the bias gradient.
template <int NP>
__global__ __launch_bounds__(256) void dig_conv_bw_merge_kernel(DigConvBwArgs a) {
    constexpr int L = dig_limbs<NP>();
    if (__builtin_amdgcn_readfirstlane(a.info->np) != a.np) return;
    __shared__ uint32_t sum[L + 1][8][33];
    const int64_t MN = (int64_t)a.M * a.N;
    const int t = threadIdx.x, o = t & 31, zl = t >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + o;
    const bool live = i < MN;
    const int m = live ? (int)(i / a.N) : 0, n = live ? (int)(i - (int64_t)m * a.N) : 0;
    uint32_t q[L], nar = 0;
#pragma unroll
    for (int l = 0; l < L; ++l) q[l] = 0;
    if (live) {
#pragma unroll 4
        for (int z = zl; z < a.splits; z += 8) {
            uint32_t p[L];
#pragma unroll
            for (int l = 0; l < L; ++l) p[l] = a.part[((int64_t)z * L + l) * MN + i];
            quire_merge<L>(q, p);
            nar |= a.rowflag[(int64_t)z * a.M + m] | a.colflag[(int64_t)z * a.N + n];
        }
    }
#pragma unroll
    for (int l = 0; l < L; ++l) sum[l][zl][o] = q[l];
    sum[L][zl][o] = nar;
    __syncthreads();
    if (zl != 0 || !live) return;
#pragma unroll
    for (int k = 1; k < 8; ++k) {
        uint32_t p[L];
#pragma unroll
        for (int l = 0; l < L; ++l) p[l] = sum[l][k][o];
        quire_merge<L>(q, p);
        nar |= sum[L][k][o];
    }
    DigRound rd;
    rd.fin = a.fin;
    rd.fout = a.fout;
    rd.at = a.info->base[0] + a.info->base[1];
    const int bits = a.qbits - rd.at;
    if (bits < 32 * L) dig_wrap<L>(q, bits);
    const uint32_t v = dig_round<L>(q, rd, nar != 0, false, 0u);
    if (n < a.crs) dig_store_pattern(a.dw, (int64_t)m * a.crs + n, rd.fout.n, v);
    else dig_store_pattern(a.dbias, m, rd.fout.n, v);
}

template <int NP>
inline hipError_t launch_dig_conv_bw_product(hipStream_t stream, DigConvBwArgs a, const DigConvBwPlan& p, uint8_t* part) {
    constexpr int L = dig_limbs<NP>();
    a.part = (uint32_t*)part;
    a.rowflag = a.part + (size_t)p.splits * L * p.M * p.N;
    a.colflag = a.rowflag + (size_t)p.splits * p.M;
    const int tc = p.WY == 1 ? DigConvShape<1>::TC : DigConvShape<2>::TC;
    const dim3 grid((unsigned)(p.tiles_m * ((p.N + tc - 1) / tc)), (unsigned)p.splits);
    if (p.WY == 1) hipLaunchKernelGGL((dig_conv_bw_kernel<NP, 1>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((dig_conv_bw_kernel<NP, 2>), grid, dim3(256), 0, stream, a);
    PNN_CHECK_LAUNCH();
    hipLaunchKernelGGL(dig_conv_bw_merge_kernel<NP>, dim3((unsigned)(((int64_t)p.M * p.N + 31) / 32)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// workspace: [planes of dy][planes of x][blocks of ones][256 zeros][decision][scan][partial sums and flags of the slices]
template <class F>
inline hipError_t launch_dig_conv_bw(hipStream_t stream, const DigConvBwPlan& p, const void* dy, const void* x, void* dw, void* dbias, int fout,
                                     void* workspace) {
    typedef typename Storage<F::N>::T T;
    typedef DigFormat<F> D;
    uint8_t* base = (uint8_t*)workspace;
    uint4* Ad = (uint4*)base;
    uint4* xb = (uint4*)(base + p.a_bytes);
    uint4* ones = (uint4*)(base + p.a_bytes + p.x_bytes);
    uint4* zero = (uint4*)(base + p.a_bytes + p.x_bytes + p.ones_bytes);
    DigInfo* info = (DigInfo*)(zero + 16);
    void* stats = (void*)(zero + 32);
    const ConvGeom& g = p.g;
    const int64_t planes = (int64_t)g.C * g.H * g.W, nx = planes * g.N, ny = (int64_t)g.N * g.K * g.OH * g.OW;
    const DigStatJob sx{x, 1, nx, nx, p.N > p.crs ? 1 : 0}, sy{dy, 1, ny, ny, 0};
    hipLaunchKernelGGL((dig_stat_kernel<F, false>), dim3((unsigned)dig_stat_wgs<false>(), 2), dim3(1024), 0, stream, sx, sy, stats);
    PNN_CHECK_LAUNCH();
    constexpr int POS = dig_bw_positions<F>(), PX = 4 / (int)sizeof(T);
    const int posmax = (2 * p.KB + p.NG - 1) / p.NG;  // positions up to the padded end of the reduction
    const int chunks = (posmax + POS - 1) / POS;
    const unsigned ablocks = (unsigned)p.RBA * (unsigned)p.NG * (unsigned)chunks;
    if (planes % PX == 0 && ((uintptr_t)x & 3u) == 0) {
        const unsigned xblocks = (unsigned)((planes / PX * p.NG + 255) / 256);
        hipLaunchKernelGGL((dig_conv_bw_digits_kernel<F, PX>), dim3(ablocks + xblocks), dim3(256), 0, stream, (const T*)dy, (const T*)x, p, Ad, xb, ones, zero,
                           ablocks, chunks, stats, info);
    } else {
        const unsigned xblocks = (unsigned)((planes * p.NG + 255) / 256);
        hipLaunchKernelGGL((dig_conv_bw_digits_kernel<F, 1>), dim3(ablocks + xblocks), dim3(256), 0, stream, (const T*)dy, (const T*)x, p, Ad, xb, ones, zero,
                           ablocks, chunks, stats, info);
    }
    PNN_CHECK_LAUNCH();
    DigConvBwArgs a;
    a.Ad = Ad; a.xb = xb; a.ones = ones; a.zero = zero; a.info = info;
    a.RBA = p.RBA; a.kb_per_split = p.kb_per_split;
    a.NG = p.NG; a.OH = g.OH; a.OW = g.OW; a.H = g.H; a.W = g.W; a.R = g.R; a.S = g.S; a.ph = g.ph; a.pw = g.pw; a.sh = g.sh; a.sw = g.sw;
    a.crs = p.crs; a.M = p.M; a.N = p.N;
    a.tiles_m = p.tiles_m;
    a.splits = p.splits;
    a.dw = dw; a.dbias = dbias;
    a.fin = fmt_of_code(code_of<F>());
    a.fout = fmt_of_code(fout);
    a.qbits = F::QBITS;
    if constexpr (D::NP1 == 4) {
        a.np = 4;
        const hipError_t e = launch_dig_conv_bw_product<4>(stream, a, p, base + p.part_off());
        if (e != hipSuccess) return e;
    }
    a.np = D::NP2;
    return launch_dig_conv_bw_product<dig_conv_wide<F>()>(stream, a, p, base + p.part_off());
}

}  // namespace pnn
