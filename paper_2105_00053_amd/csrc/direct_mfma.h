// Products and convolutions straight from the patterns on the integer matrix cores (paper Sec. 2, Sec. 3.1, Sec. 3.3): one
// launch, no rewritten operands, no scan.  For the sizes at which a call's time is its launches and the latency of one pass
// over its operands, and for the passes that no other matrix-core kernel takes (thin matrices, strided backward-data, layers
// of few channels).
//
// In units of minpos a posit is an integer of 2 MAXS + 1 bits.  Written in balanced base-256 digits, as many as the whole
// format needs (DirectFormat::NP: 2 for posit<8,0> to 8 for posit<16,1> and 11 for posit(12,2)), a product is
//     a b = sum_s 256^s sum_{i + j = s} a_i b_j :
// 2 NP - 1 int32 sums per output, exact for up to DIRECT_MAXK reduction indices (dig_planes.h).  The window is the format, so
// nothing has to be known about the data.  The sums meet in LDS as 64-bit words of four sums each, one thread combines an
// output's words modulo 2^QBITS -- the quire's limbs, wrap-around included -- and rounds once.
//
// A wave multiplies 16 x 16 outputs over every KG-th k block of 64 reduction indices: it loads the 16 consecutive indices a lane of
// v_mfma_i32_16x16x64_i8 holds of one row (lane l: row l % 16, indices 16 (l / 16) ..), turns them into digits in registers and multiplies
// all pairs of planes.  The waves of a workgroup share one tile and cut the reduction, so no pattern is converted twice in a workgroup and the
// main loop has no barrier (direct_shared_kernel: 32 x 32 outputs, planes exchanged through LDS, half the conversions and a barrier per
// step: 512^3, posit(10,1), 8.9 us against 9.4, posit<16,1> 16.4 and 22.3).
//
// What bounds it is the conversion of 32 patterns per lane and k block, about 30 vector instructions each, against NP^2 matrix
// instructions of 16 cycles; formats of up to 12 bits read a table in LDS instead that every workgroup builds (posit(12,1), 512^3 20.3 us
// by instructions, 13.0 by the table; 48 x 368 x 340 8.2 and 6.9; posit<16,1>, whose table does not fit, 22.3 and 8.7).  Whole calls,
// against the kernels on the vector ALU or with operands rewritten first: posit<16,1> 48 x 368 x 340 161 -> 8.4 us, posit(12,1) 104 -> 5.8,
// 333 x 777 x 555 22.5 -> 18.7, posit<8,0> 512^3 15.8 -> 6.1, posit(12,2) 512^3 90 -> 28.  Operands are converted once per 16 rows of the other
// side: from some 2^27 multiply-adds on (16 bits) those written once win.
#pragma once

#include "dig_planes.h"
#include "direct_gemm.h"

namespace pnn {

typedef int dm_v4i __attribute__((ext_vector_type(4)));

template <class F>
struct DirectFormat {
    static constexpr int BITS = 2 * F::MAXS + 1;
    static constexpr int NP = (BITS + 2 + 7) / 8;  // digits of the largest magnitude
    static constexpr int ND = (NP + 3) / 4;        // 32-bit words that hold them
    static constexpr int NC = 2 * NP - 1;          // sums
    static constexpr int NW = (NC + 3) / 4;        // 64-bit words of four sums
    static constexpr bool TABLE = F::N <= 12;      // digits looked up in LDS
    static constexpr int TW = ND == 3 ? 4 : ND;    // words of an entry
    static constexpr int L = Arith<F>::L;          // limbs of an output
};
// posit<32,2>: the 62 bits that eight planes hold, from the lowest bit of the workgroup's operands up (direct_p32_kernel)
template <>
struct DirectFormat<P32> {
    static constexpr int NP = 8, ND = 2, NC = 15, NW = 4, TW = 2, L = 5;
    static constexpr bool TABLE = false;
};

#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ int direct_run(uint32_t y) {  // leading bits that are alike; -1 if all are
    int n;
    asm("v_ffbh_i32 %0, %1" : "=v"(n) : "v"(y));
    return n;
}
#else
inline int direct_run(uint32_t y) {
    const uint32_t x = (int32_t)y < 0 ? ~y : y;
    return x ? __builtin_clz(x) : -1;
}
#endif

// The magnitude of a pattern (NaR: F::NAR) as an integer in units of minpos 2^base, lowest word first; zero and NaR: zero.
template <class F>
PNN_HD void direct_magnitude(uint32_t mag, uint32_t (&m)[DirectFormat<F>::ND], int base = 0) {
    constexpr int ND = DirectFormat<F>::ND;
    const uint32_t y = mag << (33 - F::N);  // first regime bit in bit 31; NaR: nothing left
    const int c = (int)y >> 31;
    const int run = direct_run(y);
    const uint32_t z = y << (run & 31);     // the bit that ended the run on top
    const uint32_t sig = ((z << F::ES) & 0x7FFFFFFFu) | ((y < 1u ? y : 1u) << 31);
    const int e = F::ES ? (int)((z >> (31 - F::ES)) & ((1u << F::ES) - 1u)) : 0;
    const int k = (run ^ ~c) + 2 * c + 1;   // run - 1 for ones, -run for zeros
    const int h = k * (1 << F::ES) + e + F::MAXS - base;  // where the leading bit belongs
    if constexpr (ND == 1) {
        m[0] = sig >> ((31 - h) & 31);
    } else if constexpr (ND == 2) {
        const uint64_t v = ((uint64_t)sig << 32) >> ((63 - h) & 63);
        m[0] = (uint32_t)v;
        m[1] = (uint32_t)(v >> 32);
    } else {
        const int t = (95 - h) & 127;  // right shift from the top of 96 bits
        const uint64_t v = ((uint64_t)sig << 32) >> (t & 31);
        const uint32_t vh = (uint32_t)(v >> 32), vl = (uint32_t)v;
        m[2] = t < 32 ? vh : 0u;
        m[1] = t < 32 ? vl : t < 64 ? vh : 0u;
        m[0] = t < 32 ? 0u : t < 64 ? vl : vh;
    }
}

// The balanced digits of a magnitude with a sign (0 or all ones): byte by byte (v + 0x80..80) ^ 0x80..80.
template <int ND>
PNN_HD void direct_balance(const uint32_t (&m)[ND], uint32_t sg, uint32_t (&d)[ND]) {
    constexpr uint32_t B = 0x80808080u;
    unsigned carry = 0;
    d[0] = __builtin_addc(m[0] ^ sg, B - sg, 0u, &carry) ^ B;
#pragma unroll
    for (int i = 1; i < ND; ++i) d[i] = __builtin_addc(m[i] ^ sg, B, carry, &carry) ^ B;
}

template <class F>
PNN_HD void direct_digits(uint32_t p, uint32_t (&d)[DirectFormat<F>::ND], int base = 0) {
    const int s = (int)(p << (32 - F::N)) >> (32 - F::N);
    uint32_t m[DirectFormat<F>::ND];
    direct_magnitude<F>(s < 0 ? 0u - (uint32_t)s : (uint32_t)s, m, base);
    direct_balance(m, (uint32_t)(s >> 31), d);
}

// ---- operands: the 16 patterns of one row from reduction index k0 on; zero from kend on ----
//
// A row index beyond the operand's rows stands for its last row: such outputs are not stored.  Offsets are 32 bits (DIRECT_EXTENT).

// 16 patterns as they lie in memory: four or two to a word
template <class T>
struct DirectRaw {
    static constexpr int PER = 4 / (int)sizeof(T);
    uint32_t w[16 / PER];
    template <class F>
    __device__ __forceinline__ uint32_t get(int i) const { return (w[i / PER] >> (8 * (int)sizeof(T) * (i % PER))) & F::MASK; }
    template <class At>  // at(i): pattern i
    __device__ __forceinline__ void gather(const At& at) {
        T v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = at(i);
#pragma unroll
        for (int i = 0; i < 16 / PER; ++i) {
            w[i] = v[PER * i];
#pragma unroll
            for (int e = 1; e < PER; ++e) w[i] |= (uint32_t)v[PER * i + e] << (8 * (int)sizeof(T) * e);
        }
    }
};

template <class T>
struct DirectMatrix {
    static constexpr bool RAISES_NAR = true;
    const T* p;
    uint32_t s_r, s_k;  // element (row, k) s_r row + s_k k bytes from p; one of the two is an element's size
    int rows;
    typedef uint32_t Row;
    __device__ __forceinline__ Row row(int r) const { return (uint32_t)(r < rows ? r : rows - 1) * s_r; }
    __device__ __forceinline__ const T* at(uint32_t bytes) const { return (const T*)((const char*)p + bytes); }
    __device__ __forceinline__ T one(Row r, int k) const { return *at(r + (uint32_t)k * s_k); }
    __device__ __forceinline__ void fetch(Row r, int k0, int kend, DirectRaw<T>& raw) const {
        if (s_k == sizeof(T) && k0 + 16 <= kend) {
            __builtin_memcpy(raw.w, at(r + (uint32_t)k0 * (uint32_t)sizeof(T)), 16 * sizeof(T));  // any alignment
            return;
        }
        const int last = kend - 1;
        raw.gather([&](int i) {
            const T v = *at(r + (uint32_t)(k0 + i < last ? k0 + i : last) * s_k);
            return k0 + i < kend ? v : (T)0;
        });
    }
};

// One fragment: 16 patterns per lane to NP planes of 16 bytes.
template <class F>
struct DirectFrag {
    typedef DirectFormat<F> D;
    typedef DirectRaw<typename Storage<F::N>::T> Raw;
    typedef uint32_t Entry __attribute__((ext_vector_type(D::TW)));
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    dm_v4i pl[D::NP];
    // nar: whether a NaR was among the patterns, as is_nar() reads it
    static constexpr uint32_t NO_NAR = F::N == 8 || F::N == 32 ? 0u : 0xFFFFFFFFu;
    __device__ static __forceinline__ bool is_nar(uint32_t nar) { return F::N == 8 || F::N == 32 ? nar != 0 : (nar & 0xFFFFu) == 0 || nar >> 16 == 0; }
    __device__ __forceinline__ void convert(const Raw& raw, const Entry* tab, uint32_t& nar, int base = 0) {
#pragma unroll
        for (int i = 0; i < 16 / Raw::PER; ++i) {
            if constexpr (F::N == 8) nar |= nar_bytes(raw.w[i]);
            else if constexpr (F::N == 32) nar |= raw.w[i] == F::NAR ? 1u : 0u;
            else nar = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, nar),
                                                                              __builtin_bit_cast(u16x2, (raw.w[i] & (F::MASK * 0x10001u)) ^ (F::NAR * 0x10001u))));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t d[4][D::ND];
            Raw in = raw;
#pragma unroll
            for (int i = 4 * q / Raw::PER; i < (4 * q + 4) / Raw::PER; ++i) asm volatile("" : "+v"(in.w[i]));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t p = in.template get<F>(4 * q + e);
                if constexpr (D::TABLE) {
                    const Entry v = tab[p];
                    if constexpr (D::TW == 1) d[e][0] = v[0];
                    else {
#pragma unroll
                        for (int h = 0; h < D::ND; ++h) d[e][h] = v[h];
                    }
                } else {
                    direct_digits<F>(p, d[e], base);
                }
            }
#pragma unroll
            for (int h = 0; h < D::ND; ++h) {  // 4 x 4 bytes transposed
                const uint32_t x = __builtin_amdgcn_perm(d[1][h], d[0][h], 0x05010400u), y = __builtin_amdgcn_perm(d[3][h], d[2][h], 0x05010400u);
                const uint32_t z = __builtin_amdgcn_perm(d[1][h], d[0][h], 0x07030602u), u = __builtin_amdgcn_perm(d[3][h], d[2][h], 0x07030602u);
                pl[4 * h][q] = (int)__builtin_amdgcn_perm(y, x, 0x05040100u);
                if (4 * h + 1 < D::NP) pl[4 * h + 1 < D::NP ? 4 * h + 1 : 0][q] = (int)__builtin_amdgcn_perm(y, x, 0x07060302u);
                if (4 * h + 2 < D::NP) pl[4 * h + 2 < D::NP ? 4 * h + 2 : 0][q] = (int)__builtin_amdgcn_perm(u, z, 0x05040100u);
                if (4 * h + 3 < D::NP) pl[4 * h + 3 < D::NP ? 4 * h + 3 : 0][q] = (int)__builtin_amdgcn_perm(u, z, 0x07060302u);
            }
            if (!D::TABLE) __builtin_amdgcn_sched_barrier(0);  // four patterns in flight: all sixteen at once take twice the registers
        }
#pragma unroll
        for (int i = 0; i < D::NP; ++i) asm volatile("" : "+v"(pl[i]));  // here, and not where they are used
    }
};

// All pairs of planes; the order keeps a sum from following itself.
template <class F>
__device__ __forceinline__ void direct_mma(const dm_v4i (&a)[DirectFormat<F>::NP], const dm_v4i (&b)[DirectFormat<F>::NP], dm_v4i (&acc)[DirectFormat<F>::NC]) {
    constexpr int NP = DirectFormat<F>::NP;
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int jj = 0; jj < NP; ++jj) {
            const int j = (i & 1) ? NP - 1 - jj : jj;
            acc[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i + j], 0, 0, 0);
        }
}

// ---- where an output goes: rows or columns contiguous in memory decide which of them neighbouring threads take ----

template <class Out> struct DirectRowsFast { static constexpr bool value = false; };
template <> struct DirectRowsFast<NchwOut> { static constexpr bool value = true; };

// LDS of a workgroup of TR x TC outputs
template <class F, int TR, int TC>
struct DirectLds {
    typedef DirectFormat<F> D;
    unsigned long long sums[D::NW][TR * TC];  // slot (block of 16 x 16, r, lane): register r of a result is row 4 (l / 16) + r, column l % 16
    uint32_t rown[TR], coln[TC];
    typename DirectFrag<F>::Entry tab[D::TABLE ? 1 << F::N : 1];
    template <int THREADS>
    __device__ __forceinline__ void clear(int t) {
        for (int i = t; i < D::NW * TR * TC; i += THREADS) (&sums[0][0])[i] = 0;
        for (int i = t; i < TR; i += THREADS) rown[i] = 0;
        for (int i = t; i < TC; i += THREADS) coln[i] = 0;
        if constexpr (D::TABLE) {
            for (int i = t; i < 1 << (F::N - 1); i += THREADS) {  // patterns of both signs from one magnitude; i = 0: zero and NaR
                uint32_t m[D::ND], d[D::ND];
                direct_magnitude<F>((uint32_t)i, m);
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    typename DirectFrag<F>::Entry v = {};
                    direct_balance(m, n ? 0xFFFFFFFFu : 0u, d);
#pragma unroll
                    for (int h = 0; h < D::ND; ++h) v[h] = d[h];
                    tab[n == 0 ? i : i == 0 ? (int)F::NAR : (1 << F::N) - i] = v;
                }
            }
        }
    }
    __device__ __forceinline__ void add(const dm_v4i (&acc)[D::NC], int block, int lane) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int x = 0; x < D::NW; ++x) {
                int64_t v = acc[4 * x][r];
                if (4 * x + 1 < D::NC) v += (int64_t)acc[4 * x + 1 < D::NC ? 4 * x + 1 : 0][r] * 256;
                if (4 * x + 2 < D::NC) v += (int64_t)acc[4 * x + 2 < D::NC ? 4 * x + 2 : 0][r] * 65536;
                if (4 * x + 3 < D::NC) v += (int64_t)acc[4 * x + 3 < D::NC ? 4 * x + 3 : 0][r] * 16777216;
                __hip_atomic_fetch_add(&sums[x][(block * 4 + r) * 64 + lane], (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
    }
};

// Outputs of a workgroup from the sums in LDS: combined, rounded and stored, or left for the merge of the slices.
template <class F, class Out, int TR, int TC, int THREADS>
__device__ __forceinline__ void direct_finish(const DirectLds<F, TR, TC>& s, const Out& out, int m0, int n0, int M, int N,
                                              const typename Storage<F::N>::T* __restrict__ bias, void* __restrict__ C, int fout, const SplitWs& ws, int at = 0) {
    typedef DirectFormat<F> D;
    constexpr int OUTS = TR * TC, L = D::L, RB = TC / 16;
    const int qfrac = F::QFRAC - at;  // the sums count units of minpos^2 2^at
    const int t = threadIdx.x;
    const bool sliced = gridDim.z > 1;
    const int64_t z = blockIdx.z;
    const FmtRT fo = fmt_of_code(fout);
    for (int o = t; o < OUTS; o += THREADS) {
        const int lr = DirectRowsFast<Out>::value ? o % TR : o / TC, lc = DirectRowsFast<Out>::value ? o / TR : o % TC;
        const int m = m0 + lr, n = n0 + lc;
        if (m >= M || n >= N) continue;
        const int slot = (((lr >> 4) * RB + (lc >> 4)) * 4 + (lr & 3)) * 64 + 16 * ((lr >> 2) & 3) + (lc & 15);
        uint32_t q[L];  // word x in units of 2^(32 x), modulo 2^(32 L)
        int64_t carry = 0;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            if (l < D::NW) carry += (int64_t)s.sums[l < D::NW ? l : 0][slot];
            q[l] = (uint32_t)carry;
            carry >>= 32;
        }
        if (sliced) {
#pragma unroll
            for (int l = 0; l < L; ++l) ws.limbs[((z * M + m) * (int64_t)N + n) * L + l] = q[l];
            continue;
        }
        bool nar = (s.rown[lr] | s.coln[lc]) != 0;
        if constexpr (F::N <= 16) {
            if (bias) {
                const uint32_t bp = bias[n];
                if (bp == F::NAR) nar = true;
                else Arith<F>::add_value(q, Arith<F>::stage(bp));
            }
        }
        const uint32_t v = fo.n <= 16 ? dig_round_limbs<L, false>(q, qfrac, fo) : dig_round_limbs<L, true>(q, qfrac, fo);
        int64_t index;
        void* dst = merge_dest(out, C, m, n, index);
        dig_store_pattern(dst, index, fo.n, nar ? fo.nar() : v);
    }
    if (sliced) {
        // as in quire_gemm_kernel: the first tile column stores the row flags, the first tile row the column flags, all of them
        if (n0 == 0)
            for (int i = t; i < TR; i += THREADS)
                if (m0 + i < M) ws.rowflag[z * M + m0 + i] = s.rown[i];
        if (m0 == 0)
            for (int i = t; i < TC; i += THREADS)
                if (n0 + i < N) ws.colflag[z * N + n0 + i] = s.coln[i];
    }
}

// MT x KG waves: wave w one block of 16 x 16 of a column of MT blocks, every KG-th k block of the reduction.
template <class F, class OpA, class OpB, class Out, int MT, int KG>
__global__ __launch_bounds__(64 * MT * KG) void direct_kernel(OpA opa, OpB opb, Out out, int M, int N, int K, int k_per_split,
                                                              const typename Storage<F::N>::T* __restrict__ bias, void* __restrict__ C, int fout,
                                                              SplitWs ws, int tiles_n) {
    typedef DirectFormat<F> D;
    constexpr int TR = 16 * MT, TC = 16, THREADS = 64 * MT * KG;
    __shared__ DirectLds<F, TR, TC> lds;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), mt = w / KG, kg = w % KG;
    const int m0 = (int)(blockIdx.x / (unsigned)tiles_n) * TR, n0 = (int)(blockIdx.x % (unsigned)tiles_n) * TC;
    const int kbeg = (int)blockIdx.z * k_per_split, kend = kbeg + k_per_split < K ? kbeg + k_per_split : K;
    const int nkb = kend > kbeg ? (kend - kbeg + 63) / 64 : 0;
    const typename OpA::Row ra = opa.row(m0 + 16 * mt + (lane & 15));
    const typename OpB::Row rb = opb.row(n0 + (lane & 15));
    lds.template clear<THREADS>(t);
    __syncthreads();
    dm_v4i acc[D::NC];
#pragma unroll
    for (int s = 0; s < D::NC; ++s) acc[s] = dm_v4i{0, 0, 0, 0};
    uint32_t na = DirectFrag<F>::NO_NAR, nb = DirectFrag<F>::NO_NAR;
    for (int kb = kg; kb < nkb; kb += KG) {
        const int k0 = kbeg + kb * 64 + 16 * (lane >> 4);
        typename DirectFrag<F>::Raw fa, fb;
        opb.fetch(rb, k0, kend, fb);
        opa.fetch(ra, k0, kend, fa);
        DirectFrag<F> a, b;
        b.convert(fb, lds.tab, nb);
        a.convert(fa, lds.tab, na);
        direct_mma<F>(a.pl, b.pl, acc);
    }
    if (kg < nkb) {
        if (OpA::RAISES_NAR && DirectFrag<F>::is_nar(na)) lds.rown[16 * mt + (lane & 15)] = 1;
        if (OpB::RAISES_NAR && DirectFrag<F>::is_nar(nb)) lds.coln[lane & 15] = 1;
        lds.add(acc, mt, lane);
    }
    __syncthreads();
    direct_finish<F, Out, TR, TC, THREADS>(lds, out, m0, n0, M, N, bias, C, fout, ws);
}

// The same for 32 x 32 outputs, every pattern converted once per workgroup: KG groups of four waves, a group takes every KG-th k
// block, each of its waves converts one of the block's four fragments into LDS and multiplies one 16 x 16 block.
template <class F, class OpA, class OpB, class Out, int KG>
__global__ __launch_bounds__(256 * KG) void direct_shared_kernel(OpA opa, OpB opb, Out out, int M, int N, int K, int k_per_split,
                                                                 const typename Storage<F::N>::T* __restrict__ bias, void* __restrict__ C, int fout,
                                                                 SplitWs ws, int tiles_n) {
    typedef DirectFormat<F> D;
    constexpr int TR = 32, TC = 32, THREADS = 256 * KG, NP = D::NP, BUFS = KG == 1 && sizeof(DirectLds<F, TR, TC>) + 2 * 4096 * NP <= 163840 ? 2 : 1;
    __shared__ DirectLds<F, TR, TC> lds;
    __shared__ dm_v4i planes[BUFS][KG][4][NP][64];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), f = w & 3, kg = w >> 2;
    const int m0 = (int)(blockIdx.x / (unsigned)tiles_n) * TR, n0 = (int)(blockIdx.x % (unsigned)tiles_n) * TC;
    const int kbeg = (int)blockIdx.z * k_per_split, kend = kbeg + k_per_split < K ? kbeg + k_per_split : K;
    const int nkb = kend > kbeg ? (kend - kbeg + 63) / 64 : 0, steps = (nkb + KG - 1) / KG;
    const typename OpA::Row ra = opa.row(m0 + 16 * f + (lane & 15));
    const typename OpB::Row rb = opb.row(n0 + 16 * (f - 2) + (lane & 15));  // of use to waves 2 and 3
    DirectRaw<typename Storage<F::N>::T> raw;
    auto fetch = [&](int st) {
        const int kb = st * KG + kg;
        if (kb >= nkb) return;
        const int k0 = kbeg + kb * 64 + 16 * (lane >> 4);
        if (f < 2) opa.fetch(ra, k0, kend, raw);
        else opb.fetch(rb, k0, kend, raw);
    };
    fetch(0);
    lds.template clear<THREADS>(t);
    __syncthreads();
    dm_v4i acc[D::NC];
#pragma unroll
    for (int s = 0; s < D::NC; ++s) acc[s] = dm_v4i{0, 0, 0, 0};
    uint32_t nar = DirectFrag<F>::NO_NAR;
    for (int st = 0; st < steps; ++st) {
        const bool live = st * KG + kg < nkb;
        dm_v4i(*const buf)[NP][64] = planes[st % BUFS][kg];
        DirectFrag<F> mine;
        if (live) mine.convert(raw, lds.tab, nar);
        if (BUFS == 1 && st > 0) __syncthreads();  // everyone has read the block before
        if (live) {
#pragma unroll
            for (int i = 0; i < NP; ++i) buf[f][i][lane] = mine.pl[i];
        }
        fetch(st + 1);
        __syncthreads();  // the other buffer was read before the last barrier but one of every wave
        if (live) {
            dm_v4i a[NP], b[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                a[i] = buf[f >> 1][i][lane];
                b[i] = buf[2 + (f & 1)][i][lane];
            }
            direct_mma<F>(a, b, acc);
        }
    }
    if (DirectFrag<F>::is_nar(nar)) {
        if (f < 2) {
            if (OpA::RAISES_NAR) lds.rown[16 * f + (lane & 15)] = 1;
        } else if (OpB::RAISES_NAR) {
            lds.coln[16 * (f - 2) + (lane & 15)] = 1;
        }
    }
    lds.add(acc, f, lane);
    __syncthreads();
    direct_finish<F, Out, TR, TC, THREADS>(lds, out, m0, n0, M, N, bias, C, fout, ws);
}

// posit<32,2>, 16 x 16 outputs, eight waves that share the reduction.  Which 62 bits of the format's 241 the planes hold is decided
// by the workgroup from its own rows and columns: a first pass over them takes the smallest and the largest magnitude (the weight of a
// pattern's last bit never falls when the magnitude grows).  Rows or columns that span more go to 512-bit quires in LDS as in
// p32_lds_gemm_kernel, two threads to an output.  N(0, 1), us a call with the general kernel and with this one: 64 x 128 x 400
// 333 and 12, 79 x 1024 x 96 85 and 16.4, 64 x 192 x 1248 269 and 21; with 2 % of the patterns from the whole range 329 and 40, 86 and 25, 271 and 110.
template <class Op>
__global__ __launch_bounds__(512) void direct_p32_kernel(Op opa, Op opb, int M, int N, int K, void* __restrict__ C, int64_t ldc, int fout, int tiles_n) {
    typedef P32 F;
    typedef DirectFormat<F> D;
    typedef Arith<F> AR;
    constexpr int KG = 8, THREADS = 64 * KG, T = 16, LIMBS = 18;
    __shared__ DirectLds<F, T, T> lds;
    __shared__ unsigned long long quire[LIMBS][T * T];
    __shared__ AR::Elem stage[2][T][T];
    __shared__ uint32_t low[2], high[2];  // smallest magnitude minus one (all ones: none), largest
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m0 = (int)(blockIdx.x / (unsigned)tiles_n) * T, n0 = (int)(blockIdx.x % (unsigned)tiles_n) * T;
    const int nkb = (K + 63) / 64;
    const typename Op::Row ra = opa.row(m0 + (lane & 15)), rb = opb.row(n0 + (lane & 15));
    lds.template clear<THREADS>(t);
    if (t < 2) {
        low[t] = 0xFFFFFFFFu;
        high[t] = 0;
    }
    __syncthreads();
    uint32_t na = 0, nb = 0, lo[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, hi[2] = {0u, 0u};
    auto scan = [&](const DirectRaw<uint32_t>& raw, uint32_t& l, uint32_t& h) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t p = raw.w[i], m = (int)p < 0 ? 0u - p : p;  // NaR stays
            l = m - 1u < l ? m - 1u : l;
            h = (m & 0x7FFFFFFFu) > h ? (m & 0x7FFFFFFFu) : h;
        }
    };
    for (int kb = w; kb < nkb; kb += KG) {
        const int k0 = kb * 64 + 16 * (lane >> 4);
        DirectRaw<uint32_t> fa, fb;
        opb.fetch(rb, k0, K, fb);
        opa.fetch(ra, k0, K, fa);
        scan(fa, lo[0], hi[0]);
        scan(fb, lo[1], hi[1]);
    }
#pragma unroll
    for (int o = 0; o < 2; ++o) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const uint32_t l = (uint32_t)__shfl_xor((int)lo[o], d), h = (uint32_t)__shfl_xor((int)hi[o], d);
            lo[o] = l < lo[o] ? l : lo[o];
            hi[o] = h > hi[o] ? h : hi[o];
        }
        if (lane == 0) {
            atomicMin(&low[o], lo[o]);
            atomicMax(&high[o], hi[o]);
        }
    }
    __syncthreads();
    int base[2];
    bool fits = true;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const uint32_t h = __builtin_amdgcn_readfirstlane(high[o]), l = __builtin_amdgcn_readfirstlane(low[o]) + 1u;
        base[o] = h ? dig_low_bit<F>(l) : 0;
        fits = fits && (h == 0 || dig_high_bit<F>(h) + 1 - base[o] <= 62);
    }
    if (fits) {
        dm_v4i acc[D::NC];
#pragma unroll
        for (int s = 0; s < D::NC; ++s) acc[s] = dm_v4i{0, 0, 0, 0};
        for (int kb = w; kb < nkb; kb += KG) {
            const int k0 = kb * 64 + 16 * (lane >> 4);
            DirectRaw<uint32_t> fa, fb;
            opb.fetch(rb, k0, K, fb);
            opa.fetch(ra, k0, K, fa);
            DirectFrag<F> a, b;
            b.convert(fb, lds.tab, nb, base[1]);
            a.convert(fa, lds.tab, na, base[0]);
            direct_mma<F>(a.pl, b.pl, acc);
        }
        if (w < nkb) {
            if (na) lds.rown[lane & 15] = 1;
            if (nb) lds.coln[lane & 15] = 1;
            lds.add(acc, 0, lane);
        }
        __syncthreads();
        direct_finish<F, RowMajorOut, T, T, THREADS>(lds, RowMajorOut{ldc}, m0, n0, M, N, nullptr, C, fout, SplitWs{nullptr, nullptr, nullptr}, base[0] + base[1]);
        return;
    }
    for (int i = t; i < LIMBS * T * T; i += THREADS) (&quire[0][0])[i] = 0;
    const int o = t & 255, half = t >> 8, r = o >> 4, c = o & 15;  // output (r, c); staging: element (k = r, row = c) of operand `half`
    const Op& op = half ? opb : opa;
    const typename Op::Row row = op.row((half ? n0 : m0) + c);
    for (int k0 = 0; k0 < K; k0 += T) {
        const uint32_t p = k0 + r < K ? op.one(row, k0 + r) : 0u;
        __syncthreads();  // the slice before has been read; the quires are clear
        if (p == F::NAR) (half ? lds.coln : lds.rown)[c] = 1;
        stage[half][r][c] = AR::stage(p);
        __syncthreads();
#pragma unroll 2
        for (int kk = half; kk < T; kk += 2) {
            const AR::Elem a = stage[0][kk][r], b = stage[1][kk][c];
            const int64_t P = (int64_t)(int32_t)a.x * (int64_t)(int32_t)b.x;
            const int s = (int)(a.y + b.y), idx = s >> 5, off = s & 31;
            const uint64_t word = (uint64_t)P << off;
            const int64_t w2 = (P >> 32) >> (32 - off);
            unsigned long long* at = &quire[idx][o];
            __hip_atomic_fetch_add(at, (unsigned long long)(uint32_t)word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_add(at + T * T, (unsigned long long)(uint32_t)(word >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_add(at + 2 * T * T, (unsigned long long)w2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
    if (half || m0 + r >= M || n0 + c >= N) return;
    uint32_t limbs[16];
    int64_t carry = 0;
#pragma unroll
    for (int l = 0; l < 16; ++l) {
        const int64_t v = (int64_t)quire[l][o] + carry;
        limbs[l] = (uint32_t)v;
        carry = v >> 32;
    }
    round_store<QuireAccum<F>, 16>(limbs, (lds.rown[r] | lds.coln[c]) != 0, fout, C, (int64_t)(m0 + r) * ldc + n0 + c);
}

// ---- host side ----

// One launch; with slices of the reduction their partial quires go to the workspace (the layout of quire_gemm.h) and are merged by a
// second.
template <class F, class OpA, class OpB, class Out>
inline hipError_t launch_direct(hipStream_t stream, const DirectPlan& p, const OpA& a, const OpB& b, const Out& out, int M, int N, int K, const void* bias,
                                void* C, int fout, void* workspace) {
    typedef typename Storage<F::N>::T T;
    SplitWs ws{nullptr, nullptr, nullptr};
    if (p.splits > 1) {
        ws.limbs = (uint32_t*)workspace;
        ws.rowflag = ws.limbs + (size_t)p.splits * M * N * Arith<F>::L;
        ws.colflag = ws.rowflag + (size_t)p.splits * M;
    }
    const T* kbias = (const T*)(p.splits > 1 ? nullptr : bias);
    auto grid = [&](int tr, int tc) { return dim3((unsigned)((M + tr - 1) / tr) * (unsigned)((N + tc - 1) / tc), 1, (unsigned)p.splits); };
    const int n16 = (N + 15) / 16, n32 = (N + 31) / 32;
#define PNN_LAUNCH_DIRECT(MT, KG)                                                                                                              \
    hipLaunchKernelGGL((direct_kernel<F, OpA, OpB, Out, MT, KG>), grid(16 * MT, 16), dim3(64 * MT * KG), 0, stream, a, b, out, M, N, K, p.k_per_split, \
                       kbias, C, fout, ws, n16)
    if (p.variant == DIRECT_W8) PNN_LAUNCH_DIRECT(1, 8);
    else if (p.variant == DIRECT_W4) PNN_LAUNCH_DIRECT(1, 4);
    else if (p.variant == DIRECT_COL) PNN_LAUNCH_DIRECT(4, 1);
    else {
        constexpr int G = direct_shared_groups<F>();
        hipLaunchKernelGGL((direct_shared_kernel<F, OpA, OpB, Out, G>), grid(32, 32), dim3(256 * G), 0, stream, a, b, out, M, N, K, p.k_per_split, kbias, C, fout,
                           ws, n32);
    }
#undef PNN_LAUNCH_DIRECT
    PNN_CHECK_LAUNCH();
    if (p.splits > 1) return launch_split_merge<F, Out>(stream, ws, p.splits, M, N, bias, C, fout, out);
    return hipSuccess;
}

}  // namespace pnn
