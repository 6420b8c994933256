// Posit operands as planes of int8 digits for the integer matrix cores, and the read-out of the sums: what the matrix
// product (gemm_dig_mfma.h) and the convolutions (conv_dig_mfma.h) of every format other than posit<8,0> share.
//
// In units of minpos a posit is an integer v (paper Sec. 2; 2^(2 MAXS) for maxpos).  Written in balanced base-256 digits,
//     v * 2^-base = sum_i d_i 256^i,  d_i in [-128, 127],  i = 0 .. NP - 1,
// a product is  a b = 2^(base_a + base_b) sum_s 256^s sum_{i + j = s} a_i b_j : 2 NP - 1 int32 sums per output, NP^2 int8
// products per posit product, exact.  With NP 2^14 at most added to a sum per reduction index, sums of up to 16352
// indices stay below 2^31.  They are combined once per output, after the reduction, and rounded once.
//
// The window.  A tensor fills a few binades of its format: four planes hold 30 or 31 bits, a Gaussian tensor of a few million
// posit<16,1> or posit(8,2) values from its largest to its smallest.  A first launch (dig_stat_kernel) takes the largest
// and the smallest non-zero magnitude of each operand; both bits that matter follow from them, because the weight of a
// pattern's last bit never falls when the magnitude grows.  All later launches of the call read the decision (dig_decide)
// from the device, so nothing comes back to the host and the calls can be captured.  NP1 planes counted down from the
// operand's own highest bit if both operands fit; otherwise NP2 planes, from minpos up where they hold the whole format;
// for posit(8,1) and posit<32,2> NP2 planes from the highest bit.  Where that does not fit (posit<32,2> over more than 62
// bits), nothing is done and the call's older kernel, launched last, does the work.
//
// Balanced digits cost one addition: (v + 0x80..80) ^ 0x80..80, byte by byte.  In an operand with NaR |v| < 2^(8 NP - 2) keeps
// the top digit within [-64, 64], so -128 there marks NaR.
#pragma once

#include <type_traits>

#include "elementwise_fast.h"
#include "gemm_p8_mfma.h"
#include "quire_gemm.h"

namespace pnn {

template <int V>
using dig_int = std::integral_constant<int, V>;

constexpr int DIG_MAXK = 16352;      // longest reduction of one set of int32 sums: 8 digit pairs * 2^14 * K < 2^31
constexpr int DIG_STAT_WGS = 128;    // workgroups that scan one operand
constexpr size_t DIG_STAT_BYTES = 2 * DIG_STAT_WGS * 16;

struct DigStat {
    uint32_t low, high;  // smallest magnitude pattern minus one (all ones: none), largest magnitude pattern
    uint32_t nar, pad;
};

// What the launches of one call agree on: the number of planes (0: the older kernel does the work) and per operand the
// weight of digit 0 (as a power of two in minpos; may be negative) and whether NaR occurs.
struct DigInfo {
    int np;
    int base[2];
    int nar[2];
    int used[2];  // planes 0 .. used - 1 hold all digits of the operand's values; the marker of NaR is in the top one
};

// Plane counts by format.  COVER: NP2 planes hold the whole format.  posit<32,2> has no narrow variant (NP1 = 0): six planes,
// 46 bits, hold no Gaussian tensor of a million values, whose smallest ones end 2^-43 below one.
template <class F>
struct DigFormat {
    static constexpr int BITS = 2 * F::MAXS + 1;        // bits of the largest magnitude
    static constexpr int FULL = (BITS + 2 + 7) / 8;
    static constexpr bool COVER = FULL <= 8;
    static constexpr int NP2 = COVER ? FULL : 8;
    static constexpr int NP1 = !COVER ? 0 : NP2 <= 4 ? 3 : 4;
    static constexpr bool BASE0 = COVER && NP2 > 4;  // the wide kernel counts its planes from the lowest bit of the operand
};

template <int NP> struct DigWord { typedef uint64_t T; };
template <> struct DigWord<4> { typedef uint32_t T; };
template <> struct DigWord<3> { typedef uint32_t T; };

// Weight (power of two in minpos) of the last bit and of the leading bit of a magnitude pattern 1 .. maxpos.
template <class F>
PNN_HD int dig_low_bit(uint32_t mag) {
    bool neg;
    uint32_t sig;
    int sh;
    decode_fixed<F>(mag, neg, sig, sh);
    return sh;
}
template <class F>
PNN_HD int dig_high_bit(uint32_t mag) {
    int nf;
    const Real r = decode_fields<F>(mag, nf);
    return r.scale + F::MAXS;
}

// Bits of magnitude that np planes hold of an operand with this largest magnitude pattern: one more where no NaR needs the
// marker and the largest value's bytes stay within 0x7F7F..7F.  (That bit keeps a Gaussian posit(8,1) tensor, 15 bits, in two
// planes.)
template <class F>
PNN_HD int dig_capacity(uint32_t high, bool nar, int np) {
    if (high == 0) return 8 * np - 2;
    int nf;
    const uint32_t sig = 0x80000000u | (uint32_t)(decode_fields<F>(high, nf).frac >> 33);
    return !nar && sig <= 0xFEFEFE00u ? 8 * np - 1 : 8 * np - 2;
}

// low, high: smallest and largest magnitude pattern of the two operands (high 0: all zero).  narrow: the call has a kernel
// of NP1 planes.
template <class F>
PNN_HD DigInfo dig_decide(const uint32_t (&low)[2], const uint32_t (&high)[2], const uint32_t (&nar)[2], bool narrow) {
    typedef DigFormat<F> D;
    int lo[2], hi[2];
    for (int o = 0; o < 2; ++o) {
        lo[o] = high[o] ? dig_low_bit<F>(low[o]) : 0;
        hi[o] = high[o] ? dig_high_bit<F>(high[o]) : 0;
    }
    auto fits = [&](int np) {
        return hi[0] + 1 - lo[0] <= dig_capacity<F>(high[0], nar[0], np) && hi[1] + 1 - lo[1] <= dig_capacity<F>(high[1], nar[1], np);
    };
    DigInfo r;
    r.np = 0;
    if (D::NP1 != 0 && narrow && fits(D::NP1)) r.np = D::NP1;
    else if (D::BASE0 || fits(D::NP2)) r.np = D::NP2;
    for (int o = 0; o < 2; ++o) {
        r.base[o] = D::BASE0 && r.np != D::NP1 ? lo[o] : hi[o] + 1 - dig_capacity<F>(high[o], nar[o], r.np);
        r.nar[o] = nar[o] ? 1 : 0;
        r.used[o] = (hi[o] + 1 - r.base[o] + 9) / 8;  // |v| < 2^b takes ceil((b + 2) / 8) balanced digits at most
    }
    return r;
}

// The digits of a pattern as bytes, digit 0 lowest; NaR: -128 in the top one.  The leading bit goes to bit
// scale + MAXS - base, all bits of a pattern that belongs in the window stay.
template <class F, int NP>
PNN_HD typename DigWord<NP>::T dig_word(uint32_t p, int base) {
    typedef typename DigWord<NP>::T W;
    constexpr W B = (W)(0x8080808080808080ull >> (64 - 8 * NP)), MASK = (W)(~0ull >> (64 - 8 * NP));
    bool neg;
    int scale, nf;
    uint32_t fr;
    decode_core(p, F::N, F::ES, neg, scale, fr, nf);
    const uint32_t sig = 0x80000000u | (fr >> 1);
    const int h = scale + F::MAXS - base;
    W m;
    if constexpr (sizeof(W) == 4) m = sig >> ((31 - h) & 31);
    else m = ((uint64_t)sig << 32) >> ((63 - h) & 63);
    const W v = neg ? (W)0 - m : m;
    const W d = ((v + B) ^ B) & MASK;
    return p == 0 ? (W)0 : p == F::NAR ? (W)0x80 << (8 * (NP - 1)) : d;
}

// ---- scan of the operands ----

struct DigStatJob {
    const void* src;
    int64_t rows, cols, ld;  // a row-major matrix as stored
    int with_one;            // the value one takes part as well (the column of ones of a bias gradient)
};

template <class F>
struct DigScan {
    uint32_t low = 0xFFFFFFFFu, high = 0, nar = 0;
    __device__ __forceinline__ void add(uint32_t p) {
        p &= F::MASK;
        const uint32_t m = (p & F::NAR) ? (0u - p) & F::MASK : p;  // NaR stays NAR
        const uint32_t l = m - 1u;
        low = l < low ? l : low;
        const uint32_t h = m & (F::NAR - 1u);
        high = h > high ? h : high;
        nar |= (uint32_t)(p == F::NAR);
    }
    __device__ __forceinline__ void merge(uint32_t l, uint32_t h, uint32_t n) {
        low = l < low ? l : low;
        high = h > high ? h : high;
        nar |= n;
    }
};

// PACK: the matrix product of posit(8,1) keeps what a workgroup saw in 16 bits (smallest magnitude minus one, largest one, NaR),
// so that the results of DIG_STAT_WGS8 workgroups fit beside the decision.  (With 28 workgroups, 32 bits each, convolutions
// too, the scan of two 2048 x 2048 operands took 13.7 us, and the weight gradient of 256 images of 128 channels at 28 x 28 to
// 128, 1 x 1, 224; now 177.)
constexpr int DIG_STAT_WGS8 = 56;
template <class F>
constexpr bool dig_stat_packed() { return F::N == 8 && !DigFormat<F>::BASE0; }
template <bool PACK>
constexpr int dig_stat_wgs() { return PACK ? DIG_STAT_WGS8 : DIG_STAT_WGS; }

// Grid (dig_stat_wgs, 2), 1024 threads: workgroup (g, o) leaves what it saw of operand o in stats[o * wgs + g].  Bound by
// memory: four 16-byte loads in flight per thread (one: 22 us for 2 x 16 MB, 1.5 TB/s).
template <class F, bool PACK>
__global__ __launch_bounds__(1024) void dig_stat_kernel(DigStatJob job0, DigStatJob job1, void* __restrict__ stats) {
    typedef typename Storage<F::N>::T T;
    constexpr int V = 16 / (int)sizeof(T);
    const DigStatJob& job = blockIdx.y == 0 ? job0 : job1;
    const T* src = (const T*)job.src;
    const int t = threadIdx.x;
    constexpr int WGS = dig_stat_wgs<PACK>();
    const int64_t step = (int64_t)WGS * 1024, first = (int64_t)blockIdx.x * 1024 + t;
    DigScan<F> s;
    auto vec = [&](const uint4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int b = 0; b < 4 / (int)sizeof(T); ++b) s.add(w[i] >> (8 * (int)sizeof(T) * b));
    };
    const bool aligned = ((uintptr_t)src & 15u) == 0;
    if (job.ld == job.cols && aligned) {
        const int64_t n = job.rows * job.cols, nv = n / V;
        const uint4* q = reinterpret_cast<const uint4*>(src);
        int64_t i = first;
        for (; i + 3 * step < nv; i += 4 * step) {
            const uint4 v0 = q[i], v1 = q[i + step], v2 = q[i + 2 * step], v3 = q[i + 3 * step];
            vec(v0);
            vec(v1);
            vec(v2);
            vec(v3);
        }
        for (; i < nv; i += step) vec(q[i]);
        const int64_t tail = nv * V + first;
        if (tail < n) s.add(src[tail]);
    } else if (aligned && job.ld % V == 0 && job.cols % V == 0) {
        const int64_t per_row = job.cols / V, nv = job.rows * per_row;
        for (int64_t i = first; i < nv; i += step) {
            const int64_t r = i / per_row;
            vec(*reinterpret_cast<const uint4*>(src + r * job.ld + (i - r * per_row) * V));
        }
    } else {
        const int64_t n = job.rows * job.cols;
        for (int64_t i = first; i < n; i += step) {
            const int64_t r = i / job.cols;
            s.add(src[r * job.ld + (i - r * job.cols)]);
        }
    }
    if (job.with_one) s.add(F::NAR >> 1);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        s.merge((uint32_t)__shfl_xor((int)s.low, d), (uint32_t)__shfl_xor((int)s.high, d), (uint32_t)__shfl_xor((int)s.nar, d));
    __shared__ DigStat part[16];
    if ((t & 63) == 0) part[t >> 6] = DigStat{s.low, s.high, s.nar, 0};
    __syncthreads();
    if (t == 0) {
#pragma unroll
        for (int i = 1; i < 16; ++i) s.merge(part[i].low, part[i].high, part[i].nar);
        const int at = blockIdx.y * WGS + blockIdx.x;
        if constexpr (PACK) ((uint16_t*)stats)[at] = (uint16_t)((s.low < 0xFFu ? s.low : 0xFFu) | (s.high << 8) | (s.nar << 15));
        else ((DigStat*)stats)[at] = DigStat{s.low, s.high, s.nar, 0};
    }
}

// Every workgroup (256 threads) of a digit launch reads the partial results and decides; the first one stores the decision
// for the launches that follow.
template <class F, bool PACK>
__device__ __forceinline__ DigInfo dig_read_decision(const void* __restrict__ stats, DigInfo* __restrict__ info, bool narrow, bool store) {
    static_assert(DIG_STAT_WGS == 128 && DIG_STAT_WGS8 <= 128, "two waves per operand");
    constexpr int WGS = dig_stat_wgs<PACK>();
    __shared__ DigStat wave[4];
    const int t = threadIdx.x, o = t >> 7, g = t & 127;
    DigScan<F> s;
    if (g < WGS) {
        if constexpr (PACK) {
            const uint32_t v = ((const uint16_t*)stats)[o * WGS + g];
            s.merge((v & 0xFFu) == 0xFFu ? 0xFFFFFFFFu : v & 0xFFu, (v >> 8) & 0x7Fu, v >> 15);
        } else {
            const DigStat v = ((const DigStat*)stats)[o * WGS + g];
            s.merge(v.low, v.high, v.nar);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        s.merge((uint32_t)__shfl_xor((int)s.low, d), (uint32_t)__shfl_xor((int)s.high, d), (uint32_t)__shfl_xor((int)s.nar, d));
    if ((t & 63) == 0) wave[t >> 6] = DigStat{s.low, s.high, s.nar, 0};
    __syncthreads();
    uint32_t low[2], high[2], nar[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        DigScan<F> u;
        u.merge(wave[2 * k].low, wave[2 * k].high, wave[2 * k].nar);
        u.merge(wave[2 * k + 1].low, wave[2 * k + 1].high, wave[2 * k + 1].nar);
        low[k] = __builtin_amdgcn_readfirstlane(u.low + 1u);
        high[k] = __builtin_amdgcn_readfirstlane(u.high);
        nar[k] = __builtin_amdgcn_readfirstlane(u.nar);
    }
    const DigInfo r = dig_decide<F>(low, high, nar, narrow);
    if (store && t == 0) *info = r;
    return r;
}

// The planes of a block fall into groups, and a block carries one bit per group that holds anything.  A window counted from
// the highest bit puts nearly all digits into its upper planes; only the rare small values reach the lower ones.  A
// workgroup therefore multiplies the planes from some group on for every k block, straight-line and without a look at the
// bits, and goes once more over the few k blocks that hold anything below.
template <int NP>
struct DigGroups {
    static constexpr int G = NP <= 5 ? 3 : 4;
    static constexpr int start(int g) {  // first plane of group g; start(G) = NP
        return g == G ? NP : NP <= 6 ? g : g == 0 ? 0 : g + 1;
    }
};

// 16 digit words (one lane's reduction indices) to NP planes of 16 bytes: 4 x 4 byte transpositions.
template <int NP>
__device__ __forceinline__ void dig_planes_of(const typename DigWord<NP>::T (&w)[16], uint32_t (&pl)[NP][4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int h = 0; h < (NP + 3) / 4; ++h) {
            uint32_t a[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = (uint32_t)(w[4 * q + e] >> (32 * h));
            const uint32_t x = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), y = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u);
            const uint32_t z = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u), u = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
            pl[4 * h][q] = __builtin_amdgcn_perm(y, x, 0x05040100u);
            if (4 * h + 1 < NP) pl[4 * h + 1 < NP ? 4 * h + 1 : 0][q] = __builtin_amdgcn_perm(y, x, 0x07060302u);
            if (4 * h + 2 < NP) pl[4 * h + 2 < NP ? 4 * h + 2 : 0][q] = __builtin_amdgcn_perm(u, z, 0x05040100u);
            if (4 * h + 3 < NP) pl[4 * h + 3 < NP ? 4 * h + 3 : 0][q] = __builtin_amdgcn_perm(u, z, 0x07060302u);
        }
    }
}

// ---- the inner step: one k block of 32, one 32 x 32 block of outputs per wave ----

// Planes SP .. TA - 1 and SP .. TB - 1 of the two blocks a wave multiplies in a step, as operand registers.
template <int NP>
struct DigFrag {
    pm_v4i a[NP], b[NP];
    template <int SP, int TA = NP, int TB = NP>
    __device__ __forceinline__ void load(const uint4* sa, const uint4* sb) {
#pragma unroll
        for (int i = NP - 1; i >= SP; --i) {
            if (i < TB) b[i] = __builtin_bit_cast(pm_v4i, sb[i * 64]);
            if (i < TA) a[i] = __builtin_bit_cast(pm_v4i, sa[i * 64]);
        }
    }
};

// Planes IF .. IT - 1 of A against JF .. JT - 1 of B; the order keeps a sum from following itself.
template <int NP, int IF, int IT, int JF, int JT>
__device__ __forceinline__ void dig_mma(const DigFrag<NP>& f, pm_v16i (&acc)[2 * NP - 1]) {
#pragma unroll
    for (int i = IF; i < IT; ++i)
#pragma unroll
        for (int jj = JF; jj < JT; ++jj) {
            const int j = ((i - IF) & 1) ? JT - 1 - (jj - JF) : jj;
            acc[i + j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.a[i], f.b[j], acc[i + j], 0, 0, 0);
        }
}

// Calls loop(TA, TB) with the fewest planes that hold the operands' digits, four at least: 4 .. 7 each, or all NP of both.
template <int NP, class Loop>
__device__ __forceinline__ void dig_for_planes(int ua, int ub, const Loop& loop) {
    static_assert(NP == 8, "eight slots");
    auto second = [&](auto ta) {
        if (ub <= 4) loop(ta, dig_int<4>());
        else if (ub == 5) loop(ta, dig_int<5>());
        else if (ub == 6) loop(ta, dig_int<6>());
        else loop(ta, dig_int<7>());
    };
    if (ua > 7 || ub > 7) loop(dig_int<NP>(), dig_int<NP>());
    else if (ua <= 4) second(dig_int<4>());
    else if (ua == 5) second(dig_int<5>());
    else if (ua == 6) second(dig_int<6>());
    else second(dig_int<7>());
}

// The pairs of groups of which at least one lies below group g0 (ma, mb: the blocks' bits, uniform).
template <int NP, int GA, int GB>
__device__ __forceinline__ void dig_mma_below(int g0, uint32_t ma, uint32_t mb, const DigFrag<NP>& f, pm_v16i (&acc)[2 * NP - 1]) {
    typedef DigGroups<NP> D;
    if constexpr (GA < D::G) {
        if constexpr (GB < D::G) {
            if ((GA < g0 || GB < g0) && (ma & (1u << GA)) && (mb & (1u << GB)))
                dig_mma<NP, D::start(GA), D::start(GA + 1), D::start(GB), D::start(GB + 1)>(f, acc);
            dig_mma_below<NP, GA, GB + 1>(g0, ma, mb, f, acc);
        } else {
            dig_mma_below<NP, GA + 1, 0>(g0, ma, mb, f, acc);
        }
    }
}

// Launch of one workgroup of 256 threads per tile and slice (y); z counts what one dimension does not hold (2^36 outputs in tiles of 64 x 32 are 2^25 workgroups).
constexpr int64_t DIG_TILES_X = ((GRID_THREADS - 1) / 256) & ~(int64_t)7;  // whole rounds over the XCDs
inline dim3 dig_tile_grid(int64_t tiles, int slices = 1) {
    return dim3((unsigned)(tiles < DIG_TILES_X ? tiles : DIG_TILES_X), (unsigned)slices, (unsigned)((tiles + DIG_TILES_X - 1) / DIG_TILES_X));
}
// This workgroup's tile in launch order; from the number of tiles on there is none.
__device__ __forceinline__ int dig_tile_id() { return (int)(blockIdx.x + blockIdx.z * (unsigned)DIG_TILES_X); }

// Workgroup `id` of `total` in an order that gives each of the eight XCDs, which take workgroups in turn, a contiguous run, so that
// neighbours share an L2.
__device__ __forceinline__ int dig_xcd_order(int id, int total) {
    const int q = id & 7, each = total >> 3, more = total & 7;
    return q * each + (q < more ? q : more) + (id >> 3);
}

// ---- the step of two k blocks: 16 rows and 32 columns per wave, v_mfma_i32_16x16x64_i8 ----

typedef int dig_v4i __attribute__((ext_vector_type(4)));

// Lane l holds row or column l % 16 and 16 reduction indices: half (l / 16) % 2 of k block l / 32 of the pair.
template <int NP>
struct DigPair {
    dig_v4i a[NP], b[2][NP];
    template <int SP, int TA = NP, int TB = NP>
    __device__ __forceinline__ void load(const uint4* sa, const uint4* sb) {
#pragma unroll
        for (int i = TA - 1; i >= SP; --i) a[i] = __builtin_bit_cast(dig_v4i, sa[i * 64]);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = TB - 1; j >= SP; --j) b[h][j] = __builtin_bit_cast(dig_v4i, sb[j * 64 + 16 * h]);
    }
};

template <int NP, int IF, int IT, int JF, int JT>
__device__ __forceinline__ void dig_pair_mma(const DigPair<NP>& f, dig_v4i (&acc)[2][2 * NP - 1]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = IF; i < IT; ++i)
#pragma unroll
            for (int jj = JF; jj < JT; ++jj) {
                const int j = ((i - IF) & 1) ? JT - 1 - (jj - JF) : jj;  // the order keeps a sum from following itself
                acc[h][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f.a[i], f.b[h][j], acc[h][i + j], 0, 0, 0);
            }
}

// As dig_mma_below
template <int NP, int GA, int GB>
__device__ __forceinline__ void dig_pair_below(int g0, uint32_t ma, uint32_t mb, const DigPair<NP>& f, dig_v4i (&acc)[2][2 * NP - 1]) {
    typedef DigGroups<NP> D;
    if constexpr (GA < D::G) {
        if constexpr (GB < D::G) {
            if ((GA < g0 || GB < g0) && (ma & (1u << GA)) && (mb & (1u << GB)))
                dig_pair_mma<NP, D::start(GA), D::start(GA + 1), D::start(GB), D::start(GB + 1)>(f, acc);
            dig_pair_below<NP, GA, GB + 1>(g0, ma, mb, f, acc);
        } else {
            dig_pair_below<NP, GA + 1, 0>(g0, ma, mb, f, acc);
        }
    }
}

// NaR markers of the top planes
template <int NP>
__device__ __forceinline__ void dig_pair_markers(int a_nar, int b_nar, const DigPair<NP>& f, uint32_t& row_nar, uint32_t (&col_nar)[2]) {
    if (a_nar) {
#pragma unroll
        for (int q = 0; q < 4; ++q) row_nar |= pm_marker_bits((uint32_t)f.a[NP - 1][q]);
    }
    if (b_nar) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) col_nar[h] |= pm_marker_bits((uint32_t)f.b[h][NP - 1][q]);
    }
}

// A single k block: lanes below 32 take plane 2 m of the rows and plane j of the columns, the lanes above planes 2 m + 1 and j - 1, the
// same 32 indices: both products belong to sum 2 m + j.  NP (NP + 1) / 2 instructions for NP^2 products of half a pair's length, where a block of zeros
// beside it would take NP^2.  sa, sb: the block as lanes below 32 read it.
template <int NP>
__device__ __forceinline__ void dig_single_mma(const uint4* sa, const uint4* sb, int lane, int a_nar, int b_nar, uint32_t& row_nar, uint32_t (&col_nar)[2],
                                               dig_v4i (&acc)[2][2 * NP - 1]) {
    constexpr int MA = (NP + 1) / 2;
    const int hi = lane >> 5;
    const dig_v4i none = {0, 0, 0, 0};
    dig_v4i a[MA];
#pragma unroll
    for (int m = 0; m < MA; ++m) {
        const bool last = 2 * m + 1 == NP;  // no plane for the lanes above
        const dig_v4i v = __builtin_bit_cast(dig_v4i, sa[(2 * m + (last ? 0 : hi)) * 64]);
        a[m] = last && hi ? none : v;
    }
    if (a_nar && hi == ((NP - 1) & 1)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) row_nar |= pm_marker_bits((uint32_t)a[MA - 1][q]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        dig_v4i b[NP + 1];
#pragma unroll
        for (int j = 0; j <= NP; ++j) {
            const bool out = j == 0 ? hi != 0 : j == NP ? hi == 0 : false;
            const dig_v4i v = __builtin_bit_cast(dig_v4i, sb[(j == 0 ? 0 : j == NP ? NP - 1 : j - hi) * 64 + 16 * h]);
            b[j] = out ? none : v;
        }
        if (b_nar && hi) {
#pragma unroll
            for (int q = 0; q < 4; ++q) col_nar[h] |= pm_marker_bits((uint32_t)b[NP][q]);
        }
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int j = 0; j <= NP; ++j)
                if (2 * m + j <= 2 * NP - 2) acc[h][2 * m + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[m], b[j], acc[h][2 * m + j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Marker bits of a row or column: of the four lanes that hold its reduction indices
__device__ __forceinline__ uint32_t dig_pair_across(uint32_t v) {
    v |= (uint32_t)__shfl_xor((int)v, 16);
    return (v | (uint32_t)__shfl_xor((int)v, 32)) & 0x80808080u;
}

// ---- the sums as one integer ----

// Limbs that hold sum_s acc[s] 256^s: 2 NP - 2 bytes above int32 sums, and a sign.
template <int NP>
constexpr int dig_limbs() { return (8 * (2 * NP - 2) + 33 + 31) / 32; }

// Four sums at a time into 64 bits by 32 x 32 + 64 multiply-adds (the powers of 256 are hidden from the compiler, which
// would make pairs of shifts and adds of them), then the words with carries.
template <int NP, class V>
__device__ __forceinline__ void dig_combine(const V (&acc)[2 * NP - 1], int r, uint32_t (&q)[dig_limbs<NP>()]) {
    constexpr int NC = 2 * NP - 1, L = dig_limbs<NP>(), W = (NC + 3) / 4;
    int c8 = 1 << 8, c16 = 1 << 16, c24 = 1 << 24;
    asm("" : "+s"(c8), "+s"(c16), "+s"(c24));
    int64_t w[W];  // units of 2^(32 i)
#pragma unroll
    for (int i = 0; i < W; ++i) {
        int64_t v = acc[4 * i][r];
        if (4 * i + 1 < NC) v += (int64_t)acc[4 * i + 1 < NC ? 4 * i + 1 : 0][r] * c8;
        if (4 * i + 2 < NC) v += (int64_t)acc[4 * i + 2 < NC ? 4 * i + 2 : 0][r] * c16;
        if (4 * i + 3 < NC) v += (int64_t)acc[4 * i + 3 < NC ? 4 * i + 3 : 0][r] * c24;
        w[i] = v;
    }
    int64_t carry = 0;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        if (l < W) carry += w[l < W ? l : 0];  // |w| < 2^56
        q[l] = (uint32_t)carry;
        carry >>= 32;
    }
}

// Sign-extends the integer from bit `bits` - 1 (bits < 32 L): the wrap of a quire that a long reduction left.
template <int L>
PNN_HD void dig_wrap(uint32_t (&q)[L], int bits) {
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const int top = bits - 1 - 32 * l;  // the sign bit, seen from this limb
        if (top >= 0 && top < 31) {
            q[l] = (uint32_t)((int32_t)(q[l] << (31 - top)) >> (31 - top));
        } else if (top < 0) {
            q[l] = l > 0 ? (uint32_t)((int32_t)q[l > 0 ? l - 1 : 0] >> 31) : 0u;
        }
    }
}

struct DigRound {
    FmtRT fin, fout;
    int at;          // base_a + base_b: weight of the sums' unit in minpos^2
    PNN_HD int qfrac() const { return 2 * fin.maxs() - at; }
};

// A multi-limb integer in units of 2^-qfrac, rounded once: the rounding of quire_to_real and encode_core as straight-line
// code, so that several outputs can be in flight in a wave (branches around each case cost most of a small product's time
// at one or two waves per SIMD).  32 or more exact bits below the leading one and whether anything lies below them
// decide the rounding of every format.  WIDE: f has more than 16 bits.
template <int L, bool WIDE>
PNN_HD uint32_t dig_round_limbs(const uint32_t (&q)[L], int qfrac, const FmtRT& f) {
    const uint32_t s = (uint32_t)((int32_t)q[L - 1] >> 31);
    uint32_t a[L];
    unsigned carry = s & 1u;
#pragma unroll
    for (int l = 0; l < L; ++l) a[l] = __builtin_addc(q[l] ^ s, 0u, carry, &carry);
    // x: the highest limb that is not zero (its bit 0 is bit `at`), y: the limb below, low: whatever lies below that
    uint32_t x = a[0], y = 0, low = 0, below = 0;
    int at = 0;
#pragma unroll
    for (int l = 1; l < L; ++l) {
        const bool up = a[l] != 0;
        x = up ? a[l] : x;
        y = up ? a[l - 1] : y;
        low = up ? below : low;
        at = up ? 32 * l : at;
        below |= a[l - 1];
    }
    const bool zero = x == 0;
    const int lz = clz32(x | 1u);  // x = 0: the result is not used
    const uint64_t t = (((uint64_t)x << 32) | y) << lz;
    const int maxs = f.maxs();
    int scale = at + 31 - lz - qfrac;
    const bool over = scale >= maxs, under = scale < -maxs;
    scale = over ? maxs - 1 : under ? -maxs : scale;  // these round to maxpos / minpos with an all-ones / zero fraction
    uint64_t frac = over ? ~0ull : under ? 0ull : t << 1;
    bool sticky = over || (!under && low != 0);
    const int k = scale >> f.es;
    const uint32_t e = (uint32_t)(scale & ((1 << f.es) - 1));
    const bool pos = k >= 0;
    const int hl = (pos ? k + 2 : 1 - k) + f.es;  // 2 .. n - 1 + es
    uint32_t body;
    if constexpr (!WIDE) {  // one 32-bit word holds regime, exponent, fraction and the bits that round them
        const uint32_t fr = (uint32_t)(frac >> 32);
        sticky = sticky || (uint32_t)frac != 0;
        const uint32_t regime = pos ? (1u << ((k + 2) & 31)) - 2u : 1u;
        const uint32_t w = (((regime << f.es) | e) << (32 - hl)) | (fr >> hl);
        sticky = sticky || (fr << (32 - hl)) != 0 || (w << f.n) != 0;
        body = w >> (33 - f.n);
        body += (w >> (32 - f.n)) & 1u & ((sticky ? 1u : 0u) | body);
    } else {
        const uint64_t regime = pos ? (1ull << ((k + 2) & 63)) - 2ull : 1ull;
        const uint64_t w = (((regime << f.es) | e) << (64 - hl)) | (frac >> hl);
        sticky = sticky || (frac << (64 - hl)) != 0 || (w << f.n) != 0;
        body = (uint32_t)(w >> (65 - f.n));
        body += (uint32_t)(w >> (64 - f.n)) & 1u & ((sticky ? 1u : 0u) | body);
    }
    return zero ? 0u : s ? (0u - body) & f.mask() : body;
}

// bias * 1 in units of minpos^2 (zero for NaR, which the caller sees to); formats of at most 16 bits.
PNN_HD __int128 dig_bias_value(uint32_t bias, const FmtRT& f) {
    if (bias == 0 || bias == f.nar()) return 0;
    bool neg;
    int scale, nf;
    uint32_t fr;
    decode_core(bias, f.n, f.es, neg, scale, fr, nf);
    const uint32_t sig = (1u << nf) | (nf ? fr >> (32 - nf) : 0u);
    const __int128 v = (__int128)((unsigned __int128)sig << (scale - nf + 2 * f.maxs()));
    return neg ? -v : v;
}

// The integer of L limbs in units of minpos^2 * 2^at as a 128-bit quire (units of minpos^2), plus a bias in its units.  Formats of at
// most 16 bits, where the sums fit 128 bits: either at < 0 and the low bits are zero, or the shift stays within.
template <int L>
PNN_HD void dig_add_bias(const uint32_t (&q)[L], int at, __int128 bias, uint32_t (&out)[4]) {
    static_assert(L >= 3, "three limbs or more");
    const uint32_t top = L >= 4 ? q[L >= 4 ? 3 : 0] : (uint32_t)((int32_t)q[L - 1] >> 31);
    unsigned __int128 x = ((unsigned __int128)(((uint64_t)top << 32) | q[2]) << 64) | (((uint64_t)q[1] << 32) | q[0]);
    x = at >= 0 ? x << at : (unsigned __int128)((__int128)x >> -at);
    x += (unsigned __int128)bias;
#pragma unroll
    for (int l = 0; l < 4; ++l) out[l] = (uint32_t)(x >> (32 * l));
}

// Outputs of at most 16 bits or more, with a bias or without.  None of these sums leaves the range of its quire (at most
// 16352 terms), so there is no wrap to reproduce.
template <int L>
__device__ __forceinline__ uint32_t dig_round(const uint32_t (&q)[L], const DigRound& d, bool nar, bool has_bias, uint32_t bias) {
    uint32_t res;
    if (has_bias) {
        nar = nar || bias == d.fin.nar();
        uint32_t u[4];
        dig_add_bias<L>(q, d.at, dig_bias_value(bias, d.fin), u);
        const int qf = 2 * d.fin.maxs();
        res = d.fout.n <= 16 ? dig_round_limbs<4, false>(u, qf, d.fout) : dig_round_limbs<4, true>(u, qf, d.fout);
    } else {
        res = d.fout.n <= 16 ? dig_round_limbs<L, false>(q, d.qfrac(), d.fout) : dig_round_limbs<L, true>(q, d.qfrac(), d.fout);
    }
    return nar ? d.fout.nar() : res;
}

// ---- the same through binary64: up to four planes, formats of at most 16 bits ----
//
// The sums fall into two parts that are exact in binary64: a sum of s holds at most min(s + 1, 2 NP - 1 - s) digit pairs of
// at most 2^14 each over at most 16352 indices, so that for four planes sums 0 .. 2 stay below 2^47 and sums 3 .. 6, in
// units of 2^24, below 2^53 (with three planes: 0 and 1, 2 .. 4, less).  The parts' sum and its exact error round as in
// elementwise_fast.h: about 50 instructions per output and no pass through LDS, where the integers' way takes over 100.

// s + e = a + b exactly, s the rounded sum
PNN_HD void dig_two_sum(double a, double b, double& s, double& e) {
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// (s, e) + b: s the new rounded sum, e with the sign of the exact error and less than a unit of s's last place.  If s + b
// cancels (e1 = 0) the second sum is exact; otherwise u is below s1's last places, so r is a multiple of u's unit and v,
// half of that at most, decides the sign only where r is zero.
PNN_HD void dig_add_f64(double& s, double& e, double b) {
    double s1, e1, u, v, r;
    dig_two_sum(s, b, s1, e1);
    dig_two_sum(e1, e, u, v);
    dig_two_sum(s1, u, s, r);
    e = r + v;
}

// value of a pattern (not NaR) times 2^up; formats of at most 16 bits
PNN_HD double dig_f64_of_pattern(uint32_t p, const FmtRT& f, int up) {
    if (p == 0) return 0.0;
    bool neg;
    int scale, nf;
    uint32_t fr;
    decode_core(p, f.n, f.es, neg, scale, fr, nf);
    return f64_from_words(((uint32_t)(scale + up + 1023) << 20) | (fr >> 12) | (neg ? 0x80000000u : 0u), 0u);
}

// Constants of the rounding to a format of at most 16 bits, and the weight of the sums' unit (2^-qfrac).
struct DigF64Round {
    uint32_t minhi, maxhi, qf, himask, lomask, jam, half, mask;
    int esh, n;
    PNN_HD DigF64Round(const FmtRT& f, int qfrac) {
        const int maxs = f.maxs(), hb = f.n - 12 + f.es;
        minhi = (uint32_t)(1023 - maxs) << 20;
        maxhi = (uint32_t)(1023 + maxs) << 20;
        qf = (uint32_t)qfrac << 20;
        himask = hb > 0 ? (1u << hb) - 1u : 0u;
        lomask = hb >= 0 ? 0xFFFFFFFFu : 0xFFFFFFFFu >> -hb;
        jam = 1u << f.n;
        half = (1u << (32 - f.n)) - 1u;
        mask = f.mask();
        esh = 20 + f.es;
        n = f.n;
    }
    // s + err, rounded once (round_sum_to_body explains the steps)
    PNN_HD uint32_t operator()(double s, double err) const {
        uint32_t hi = f64_hi(s);
        const uint32_t lo = f64_lo(s), ehi = f64_hi(err);
        const bool toward_zero = (ehi ^ (hi & 0x80000000u)) > 0x80000000u;
        const uint32_t sm = (uint32_t)((int32_t)hi >> 31);
        hi -= toward_zero && lo == 0u ? 1u : 0u;
        const uint32_t ah0 = (hi & 0x7FFFFFFFu) - qf;
        const uint32_t ah = ah0 < minhi ? minhi : (ah0 > maxhi ? maxhi : ah0);
        const uint32_t h1 = ah - (1023u << 20);
        const int k = (int32_t)h1 >> esh;
        const uint32_t sg = (uint32_t)(k >> 31);
        const uint32_t kk = (uint32_t)k ^ sg;
        const uint32_t tail = funnel_shr(h1, lo, esh);
        const uint32_t below = (h1 & himask) | (lo & lomask) | (ehi << 1);
        const uint32_t w = funnel_shr(2u, (tail | (below != 0u ? jam : 0u)) ^ sg, 2);
        const uint32_t x = (uint32_t)((int32_t)w >> kk) ^ sg;
        const uint32_t lsb = (x >> (33 - n)) & 1u;
        const uint32_t body = (x + half + lsb) >> (33 - n);
        return s == 0.0 ? 0u : ((body ^ sm) - sm) & mask;
    }
};

#if defined(__HIPCC__)
template <int NP>
struct DigF64 {
    static_assert(NP == 3 || NP == 4, "parts that are exact in binary64");
    static constexpr int NC = 2 * NP - 1, LOW = NP - 1;  // sums of the low part
    template <class V>
    static __device__ __forceinline__ void parts(const V (&acc)[NC], int r, double& hi, double& lo) {
        hi = (double)acc[LOW][r] * pow2d(8 * LOW);
#pragma unroll
        for (int s = LOW + 1; s < NC; ++s) hi = __builtin_fma((double)acc[s][r], pow2d(8 * s), hi);
        lo = (double)acc[0][r];
#pragma unroll
        for (int s = 1; s < LOW; ++s) lo = __builtin_fma((double)acc[s][r], pow2d(8 * s), lo);
    }
};
#endif

__device__ __forceinline__ uint32_t dig_load_pattern(const void* p, int64_t i, int n) {
    return n <= 8 ? ((const uint8_t*)p)[i] : n <= 16 ? ((const uint16_t*)p)[i] : ((const uint32_t*)p)[i];
}
__device__ __forceinline__ void dig_store_pattern(void* p, int64_t i, int n, uint32_t v) {
    if (n <= 8) ((uint8_t*)p)[i] = (uint8_t)v;
    else if (n <= 16) ((uint16_t*)p)[i] = (uint16_t)v;
    else ((uint32_t*)p)[i] = v;
}

}  // namespace pnn
