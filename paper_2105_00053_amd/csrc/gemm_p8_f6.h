// posit<8,0> matrix product with the 32-bit quire of Table 1 (paper Sec. 2, Sec. 3.3) on the 6-bit floating-point matrix
// cores, exact.
//
// A decoded posit<8,0> v (units of minpos = 2^-6) has at most six significant bits, so for |v| < 2^11 it is the sum of two
// numbers of at most four, v = 32 h + l with h = round(v / 32), |h| <= 48 and |l| <= 16: both are integers of the 6-bit
// floating-point format E2M3 (in units of its smallest value: 0 .. 16, even to 32, multiples of four to 60).  The matrix
// instruction multiplies E2M3 by E2M3 into binary32 at twice the int8 rate, so of
//     a b = 2^10 (ah bh) + [2^5 (ah bl + al bh) + al bl]
// two binary32 sums per output are kept, HH and Q (the bracket, its products brought to one unit by the instruction's scale
// operands).  Both are sums of integers, and exact as long as the magnitudes that enter them add up to less than 2^24.
// That the instruction itself loses nothing below 2^24 was checked on the hardware against integers (random and adversarial
// digits, accumulators up to +-2^24); products of E2M3 numbers differ by a factor of at most 2^12, inside the window in which
// it aligns its products (with E3M2 on both sides ratios of 2^14 fall out of that window).
//
// The bound is proved for the whole product before anything is multiplied: the launch that writes the digits leaves, for every
// chunk of 256 reduction indices and every 128 rows, the largest sum of h^2 and of l^2 over a row; by Cauchy's inequality the
// sums stay below  sum over chunks of  |ha||hb|  and  32 (|ha||lb| + |la||hb|) + |la||lb|,  with the largest of each over all
// rows.  N(0, 1) operands with K = 4096 reach a third of 2^24.  If the bound fails, or one of the four patterns +-32, +-64 (no
// such digits) is met anywhere, every workgroup returns, and the int8 kernel of gemm_p8_mfma.h, launched behind this one, takes
// the product; otherwise that one returns at once (1.5 us a launch).
#pragma once

#include "gemm_p8_mfma.h"

namespace pnn {

typedef int pf_v8i __attribute__((ext_vector_type(8)));
typedef float pf_v16f __attribute__((ext_vector_type(16)));

constexpr int PF_UNIT = 32;          // v = PF_UNIT h + l
constexpr int PF_MAX_V = 2048;       // magnitudes from here on have no digits
constexpr int PF_CHUNK = 4;          // k blocks of 64 per chunk of the bounds
constexpr int PF_STAGES = 3;         // k blocks of 64 in LDS
constexpr int PF_MAX_K = 7168;       // beyond, ordinary data come near the bound
constexpr int PF_MIN_TILES = 256;    // fewest tiles of 128 x 128
constexpr int PF_DECIDERS = 1024;    // workgroups that work out the bound: twice what the chip holds at once
constexpr int PF_WRITERS = 8;        // of them, those that write it down (one per XCD; all of them: 12 us instead of 5 a refused launch)
constexpr float PF_LIMIT = 16776000.0f;  // a little below 2^24: the bounds are worked out in binary32
// scale operands (powers of two, bias 127) that turn E2M3 numbers, multiples of 2^-3, into integers: l, h, and h in units of l
constexpr int PF_SCALE = 127 + 3, PF_SCALE_H32 = 127 + 3 + 5;
constexpr int PF_E2M3 = 2;           // format selector of the instruction

// E2M3 code of an integer digit (units of 2^-3)
PNN_HD uint32_t pf_code(int d) {
    const int m = d < 0 ? -d : d;
    const uint32_t c = m < 16 ? (uint32_t)m : m < 32 ? 16u | (uint32_t)((m >> 1) - 8) : 24u | (uint32_t)((m >> 2) - 8);
    return d < 0 ? c | 32u : c;
}

// The integer digit of an E2M3 code (host checks)
PNN_HD int pf_value(uint32_t code) {
    const int e = (int)(code >> 3) & 3, f = (int)code & 7;
    const int m = e == 0 ? f : (8 + f) << (e - 1);
    return code & 32u ? -m : m;
}

// Digits of a decoded value with |v| < PF_MAX_V
PNN_HD void pf_split(int v, int& h, int& l) {
    const int m = v < 0 ? -v : v;
    h = (m + PF_UNIT / 2) / PF_UNIT;
    l = m - PF_UNIT * h;
    if (v < 0) { h = -h; l = -l; }
}

// Table entry of a pattern.  x: code of h in bits 0-5, of l in bits 16-21, bit 30 for NaR, bit 31 for a value without
// digits (both with zero digits).  y: l^2, and h^2 from bit 16 on.
PNN_HD uint2 pf_entry(uint32_t pattern) {
    if (pattern == 0x80u) return make_uint2(1u << 30, 0u);
    const int v = Arith<P8>::stage(pattern);
    if (v >= PF_MAX_V || v <= -PF_MAX_V) return make_uint2(1u << 31, 0u);
    int h, l;
    pf_split(v, h, l);
    return make_uint2(pf_code(h) | (pf_code(l) << 16), (uint32_t)(l * l) | ((uint32_t)(h * h) << 16));
}

struct P8F6Job {
    const uint8_t* src;
    int64_t s_r, s_k;   // element (row, k) at src[row * s_r + k * s_k]; one of the two is 1
    int rows, K;
    uint4* dst;         // [KB][RB][3][64]: per lane h[0-3]; h[4-5], l[0-1]; l[2-5] of its 32 codes of six bits each
    uint2* stat;        // [tile of 128 rows][chunk]: {largest sum of h^2 over a row, bit 31: a value has no digits; of l^2}
    uint32_t* nar;      // [tile][chunk][4]: the rows of each row block that hold NaR
    int RB, KB, chunks; // row blocks of 32 (a multiple of four), k blocks of 64
};

// Digits and bounds of both operands in one launch: the first blocks0 workgroups take job0, the rest job1.  A workgroup: four
// row blocks, one per wave, and one chunk.  Bound by memory (a byte read and 1.5 written per element: 2 x 16.7 M elements take
// 18.9 us, 4.4 TB/s), with about nine vector operations per element beside it.  A wave that has met a value without digits, which
// refuses the product, writes no more of them.
template <int UNUSED = 0>
__global__ __launch_bounds__(256) void p8_f6_digits_kernel(P8F6Job job0, P8F6Job job1, unsigned blocks0, uint32_t* verdict) {
    // One table of 256 entries and, for an operand stored reduction-index-major, one k block of 128 rows turned: rows of 72
    // bytes, 8-byte words exchanged by the row block so that neither side conflicts.
    constexpr int PITCH = 72;
    __shared__ __attribute__((aligned(16))) uint2 tab[256];
    __shared__ __attribute__((aligned(16))) uint8_t tile[128 * PITCH];
    __shared__ uint2 best[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (blockIdx.x == 0 && t == 0) *verdict = PF_UNDECIDED;
    tab[t] = pf_entry((uint32_t)t);
    __syncthreads();
    const bool first = blockIdx.x < blocks0;
    const P8F6Job& job = first ? job0 : job1;
    const unsigned lin = first ? blockIdx.x : blockIdx.x - blocks0;
    const unsigned gx = (unsigned)job.RB / 4;
    const int bx = (int)(lin % gx), chunk = (int)(lin / gx);
    const int rb = bx * 4 + wave;
    const bool via_lds = job.s_k != 1;
    const int nkb = (job.KB - chunk * PF_CHUNK) < PF_CHUNK ? (job.KB - chunk * PF_CHUNK) : PF_CHUNK;
    uint32_t raw[PF_CHUNK][8];
    if (!via_lds) {
        const int row = rb * 32 + (lane & 31);
#pragma unroll
        for (int c = 0; c < PF_CHUNK; ++c) {
            const int k0 = (chunk * PF_CHUNK + c) * 64 + 32 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 8; ++q) raw[c][q] = 0;
            if (c < nkb && row < job.rows && k0 < job.K) {
                const uint8_t* p = job.src + (int64_t)row * job.s_r + k0;
                if (k0 + 32 <= job.K) {
                    __builtin_memcpy(&raw[c][0], p, 16);  // any alignment: global memory takes 16-byte accesses at any address
                    __builtin_memcpy(&raw[c][4], p + 16, 16);
                } else {
#pragma unroll
                    for (int b = 0; b < 32; ++b)
                        if (k0 + b < job.K) raw[c][b >> 2] |= (uint32_t)p[b] << (8 * (b & 3));
                }
            }
        }
    } else {
        // thread: eight k of four consecutive rows
        const int row0 = bx * 128 + (t & 31) * 4;
        const bool rows4 = row0 + 4 <= job.rows;
#pragma unroll
        for (int c = 0; c < PF_CHUNK; ++c) {
            const int k0 = (chunk * PF_CHUNK + c) * 64 + (t >> 5) * 8;
            const uint8_t* p = job.src + (int64_t)k0 * job.s_k + row0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                raw[c][q] = 0;
                if (c < nkb && k0 + q < job.K) {
                    if (rows4) {
                        __builtin_memcpy(&raw[c][q], p + (int64_t)q * job.s_k, 4);
                    } else {
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            if (row0 + b < job.rows) raw[c][q] |= (uint32_t)p[(int64_t)q * job.s_k + b] << (8 * b);
                    }
                }
            }
        }
    }
    uint32_t hs = 0, ls = 0, flags = 0;
#pragma unroll
    for (int c = 0; c < PF_CHUNK; ++c) {
        if (c >= nkb) break;
        uint32_t w[8];
        if (via_lds) {
            if (c > 0) __syncthreads();
            const int g = t >> 5, wb = (t & 31) >> 3;  // group of eight k; row block of the thread's rows
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t d[2];
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const uint32_t* r = &raw[c][4 * half];
                    d[half] = ((r[0] >> (8 * i)) & 0xFFu) | (((r[1] >> (8 * i)) & 0xFFu) << 8) | (((r[2] >> (8 * i)) & 0xFFu) << 16) | ((r[3] >> (8 * i)) << 24);
                }
                *reinterpret_cast<uint2*>(&tile[((t & 31) * 4 + i) * PITCH + ((g ^ wb) & 7) * 8]) = make_uint2(d[0], d[1]);
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint2 v = *reinterpret_cast<const uint2*>(&tile[(wave * 32 + (lane & 31)) * PITCH + ((4 * (lane >> 5) + q) ^ wave) * 8]);
                w[2 * q] = v.x;
                w[2 * q + 1] = v.y;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) w[q] = raw[c][q];
        }
        if (__any((int)flags < 0)) continue;
        uint32_t o[12];
#pragma unroll
        for (int q = 0; q < 12; ++q) o[q] = 0;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            uint32_t sq = 0;  // 16 times l^2 <= 256 below, 16 times h^2 <= 2304 above: no carry between them, none out
#pragma unroll
            for (int bb = 0; bb < 16; ++bb) {
                const int b = part * 16 + bb;
                const uint2 e = tab[(w[b >> 2] >> (8 * (b & 3))) & 0xFFu];
                const uint32_t h = e.x & 63u, l = (e.x >> 16) & 63u;
                const int at = (6 * b) >> 5, sh = (6 * b) & 31;
                o[at] |= h << sh;
                o[6 + at] |= l << sh;
                if (sh > 26) {
                    o[at + 1] |= h >> (32 - sh);
                    o[6 + at + 1] |= l >> (32 - sh);
                }
                sq += e.y;
                flags |= e.x;
            }
            ls += sq & 0xFFFFu;
            hs += sq >> 16;
        }
        uint4* out = job.dst + ((int64_t)(chunk * PF_CHUNK + c) * job.RB + rb) * 192 + lane;
        out[0] = make_uint4(o[0], o[1], o[2], o[3]);
        out[64] = make_uint4(o[4], o[5], o[6], o[7]);
        out[128] = make_uint4(o[8], o[9], o[10], o[11]);
    }
    // lanes l and l + 32 hold the two halves of row l
    hs += (uint32_t)__shfl_xor((int)hs, 32);
    ls += (uint32_t)__shfl_xor((int)ls, 32);
    flags |= (uint32_t)__shfl_xor((int)flags, 32);
#pragma unroll
    for (int d = 1; d < 32; d *= 2) {
        const uint32_t ho = (uint32_t)__shfl_xor((int)hs, d), lo = (uint32_t)__shfl_xor((int)ls, d);
        hs = hs > ho ? hs : ho;
        ls = ls > lo ? ls : lo;
    }
    const uint64_t nar = __ballot((flags >> 30) & 1u), big = __ballot(flags >> 31);
    const int64_t at = (int64_t)bx * job.chunks + chunk;
    if (lane == 0) {
        job.nar[at * 4 + wave] = (uint32_t)nar;
        best[wave] = make_uint2(hs | (big != 0 ? 1u << 31 : 0u), ls);
    }
    __syncthreads();
    if (t == 0) {
        uint2 m = best[0];
#pragma unroll
        for (int v = 1; v < 4; ++v) {
            m.x = m.x > best[v].x ? m.x : best[v].x;
            m.y = m.y > best[v].y ? m.y : best[v].y;
        }
        job.stat[at] = m;
    }
}

struct P8F6Args {
    const uint4* Ad;
    const uint4* Bd;
    const uint2* sa;       // see P8F6Job
    const uint2* sb;
    const uint32_t* nar_a;
    const uint32_t* nar_b;
    int RBA, RBB, KB, chunks;
    const uint8_t* bias;
    void* C;
    int64_t ldc;
    int fout, M, N, tiles_m, tiles_n;
    uint32_t* verdict;     // see pf_done
};

// Operand registers of one block of 32 rows and 64 reduction indices.
struct P8F6Frag {
    pf_v8i h, l;
    // (Read as vectors: a copy of the struct would make the compiler wait for every copy in flight first.)
    __device__ __forceinline__ void load(const uint4* p) {
        const pm_v4i a = __builtin_bit_cast(pm_v4i, p[0]), b = __builtin_bit_cast(pm_v4i, p[64]), c = __builtin_bit_cast(pm_v4i, p[128]);
        h = pf_v8i{a[0], a[1], a[2], a[3], b[0], b[1], 0, 0};
        l = pf_v8i{b[2], b[3], c[0], c[1], c[2], c[3], 0, 0};
    }
};

template <int SA, int SB>
__device__ __forceinline__ pf_v16f pf_mma(const pf_v8i& a, const pf_v8i& b, const pf_v16f& c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, PF_E2M3, PF_E2M3, 0, SA, 0, SB);
}

// 128 x 128 outputs per workgroup of four waves, 64 x 64 per wave: two sums of 2 x 2 blocks, 128 registers, which leaves two waves
// per SIMD.  The product is taken transposed (columns of C along the instruction's rows): a lane then holds one row of C and,
// after exchanging halves with the lane 32 further, 16 consecutive bytes of it per block.
//
// Bound by power: the matrix instructions alone, from registers, take 84 us for 4096^3 at the 1.56 GHz the card then holds
// (int8, four products: 126 us); this kernel takes 129 us at 1.92 GHz with the matrix pipes busy half of the cycles.  Copies
// cost 14 to 20 us of that, LDS reads 14, rounding and stores 7.  Measured against it: 256 x 128 outputs with 128 x 64 per
// wave and one wave per SIMD (fewer bytes, nothing to fill the waits) 132 to 137 us, 256 x 128 with eight waves 137.
template <int UNUSED = 0>
__global__ __launch_bounds__(256, 2) void p8_f6_gemm_kernel(P8F6Args g) {
    constexpr int BI = 2, BJ = 2, WY = 2, WX = 2, W = WY * WX, THREADS = 64 * W;
    constexpr int NA = WY * BI, NB = WX * BJ;         // row and column blocks of the tile
    constexpr int RUN = 192;                          // words of 16 bytes per block of 32 x 64
    constexpr int STAGE = (NA + NB) * RUN;
    constexpr int TR = 32 * NA, TC = 32 * NB;
    constexpr int S = PF_STAGES;                      // 72 KB of LDS for each of two workgroups
    // One LDS object (beside a second one the compiler waits for every copy in front of each read of the ring)
    __shared__ uint4 lds[S * STAGE + (NA + NB + 3) / 4 + 1];
    uint32_t* const nar = reinterpret_cast<uint32_t*>(lds + S * STAGE);  // [NA + NB]: rows of each block that hold NaR
    uint32_t* const seen = nar + (NA + NB + 3) / 4 * 4;                      // the verdict as this workgroup found it
    uint4* const most = lds + (S - 1) * STAGE;                              // [THREADS], in the buffer that nothing has been copied to yet

    const int t = threadIdx.x;
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wy = w / WX, wx = w % WX;
    int tm, tn;
    pm_tile(blockIdx.x, g.tiles_m, g.tiles_n, tm, tn);

    // A k block is NA contiguous blocks of A and NB of B; a wave copies a quarter of each straight into LDS.
    constexpr int PA = NA * 3072 / W, PB = NB * 3072 / W;       // bytes per wave
    constexpr int CA = PA / 1024, CB = PB / 1024;               // copies per wave, 16 bytes per lane
    static_assert(CA * 1024 == PA && CB * 1024 == PB, "copies split evenly over the waves");
    const uint8_t* pa = (const uint8_t*)g.Ad + (int64_t)tm * NA * 3072 + w * PA;
    const uint8_t* pb = (const uint8_t*)g.Bd + (int64_t)tn * NB * 3072 + w * PB;
    const int64_t a_adv = (int64_t)g.RBA * 3072, b_adv = (int64_t)g.RBB * 3072;
    const int last = g.KB - 1;
    int next_kb = 0;
    auto issue = [&](int buf) {
        uint8_t* da = (uint8_t*)(lds + buf * STAGE) + w * PA;
        uint8_t* db = (uint8_t*)(lds + buf * STAGE + NA * RUN) + w * PB;
#pragma unroll
        for (int c = 0; c < CA; ++c)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pa + c * 1024 + lane * 16),
                                             (__attribute__((address_space(3))) void*)(da + c * 1024), 16, 0, 0);
#pragma unroll
        for (int c = 0; c < CB; ++c)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pb + c * 1024 + lane * 16),
                                             (__attribute__((address_space(3))) void*)(db + c * 1024), 16, 0, 0);
        // past the end the last block is copied again, into buffers that nothing reads: the counts of the waits stay the same
        if (next_kb < last) {
            pa += a_adv;
            pb += b_adv;
        }
        ++next_kb;
    };
    // ---- the bound, and the NaR rows of this tile ----
    // The first workgroups all work out the bound from the same numbers, a lane per chunk and eight tiles of rows side by side; one
    // that starts later looks whether they have refused by then (if it runs on all the same, the int8 kernel writes over what it
    // leaves).
    const bool decides = blockIdx.x < PF_DECIDERS;
    const int c = t & 31;
    static_assert((PF_MAX_K + 64 * PF_CHUNK - 1) / (64 * PF_CHUNK) <= 32, "a lane per chunk");
    static_assert(NA == 4 && NB == 4, "a word of NaR rows per block");
    if (t < NA + NB) nar[t] = 0;
    const int cc = c < g.chunks ? c : g.chunks - 1;
    const bool of_a = t < 32;
    uint4 rows = make_uint4(0, 0, 0, 0);
    if (t < 64) rows = *reinterpret_cast<const uint4*>(of_a ? g.nar_a + ((int64_t)tm * g.chunks + cc) * 4 : g.nar_b + ((int64_t)tn * g.chunks + cc) * 4);
    struct Most {
        uint2 a[4], b[4];
    };
    auto look = [&](Most& s, int i0) {  // past the end the last tile again
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + (t >> 5) + 8 * u;
            s.a[u] = g.sa[(int64_t)(i < g.tiles_m ? i : g.tiles_m - 1) * g.chunks + cc];
            s.b[u] = g.sb[(int64_t)(i < g.tiles_n ? i : g.tiles_n - 1) * g.chunks + cc];
        }
    };
    uint4 m = make_uint4(0, 0, 0, 0);
    auto take = [&](const Most& s) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            m.x = m.x > s.a[u].x ? m.x : s.a[u].x;
            m.y = m.y > s.a[u].y ? m.y : s.a[u].y;
            m.z = m.z > s.b[u].x ? m.z : s.b[u].x;
            m.w = m.w > s.b[u].y ? m.w : s.b[u].y;
        }
    };
    Most s0;
    if (decides) look(s0, 0);
    issue(0);
    issue(1);
    if (decides) {
        take(s0);
        for (int i = 32; i < g.tiles_m || i < g.tiles_n; i += 32) {
            look(s0, i);
            take(s0);
        }
        most[t] = c < g.chunks ? m : make_uint4(0, 0, 0, 0);
    } else if (t == 0) {
        *seen = __hip_atomic_load(g.verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(pcm_vmcnt((S - 2) * (CA + CB)));  // block 0 has landed
    __syncthreads();
    if (rows.x | rows.y | rows.z | rows.w) {
        uint32_t* const to = nar + (of_a ? 0 : NA);
        atomicOr(&to[0], rows.x);
        atomicOr(&to[1], rows.y);
        atomicOr(&to[2], rows.z);
        atomicOr(&to[3], rows.w);
    }
    bool refused;
    if (decides) {
        m = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < THREADS / 32; ++v) {
            const uint4 s = most[32 * v + c];
            m.x = m.x > s.x ? m.x : s.x;
            m.y = m.y > s.y ? m.y : s.y;
            m.z = m.z > s.z ? m.z : s.z;
            m.w = m.w > s.w ? m.w : s.w;
        }
        const float ha = __builtin_sqrtf((float)m.x), la = __builtin_sqrtf((float)m.y), hb = __builtin_sqrtf((float)m.z), lb = __builtin_sqrtf((float)m.w);
        float bhh = ha * hb + ((m.x | m.z) >> 31 ? 1e30f : 0.0f), bq = (float)PF_UNIT * (ha * lb + la * hb) + la * lb;
#pragma unroll
        for (int d = 1; d < 32; d *= 2) {
            bhh += __shfl_xor(bhh, d);
            bq += __shfl_xor(bq, d);
        }
        refused = !(bhh < PF_LIMIT / 16 && bq < PF_LIMIT);
        if (t == 0 && blockIdx.x < PF_WRITERS) __hip_atomic_store(g.verdict, refused ? PF_REFUSED : PF_DONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        refused = *seen == PF_REFUSED;
    }
    if (__builtin_amdgcn_readfirstlane(refused)) {
        __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
        return;
    }

    pf_v16f hh[BI][BJ], qq[BI][BJ];
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) hh[i][j][r] = qq[i][j][r] = 0.0f;

    struct Frags {
        P8F6Frag a[BI], b[BJ];
    };
    const uint4* const la0 = lds + wy * BI * RUN + lane;
    const uint4* const lb0 = lds + (NA + wx * BJ) * RUN + lane;
    auto load = [&](Frags& f, int buf) {
#pragma unroll
        for (int j = 0; j < BJ; ++j) f.b[j].load(lb0 + buf * STAGE + j * RUN);
#pragma unroll
        for (int i = 0; i < BI; ++i) f.a[i].load(la0 + buf * STAGE + i * RUN);
    };
    // One step: k block kb is in cur.  Before the barrier this wave's copies of block kb + 1 have landed; behind it everyone's
    // have, and everyone's reads of block kb - 1 (issued in the step before last) have been consumed, so its buffer takes a copy.
    int buf = 0;  // of the block in cur
    auto step = [&](const Frags& cur, Frags& next) {
        __builtin_amdgcn_s_waitcnt(pcm_vmcnt((S - 3) * (CA + CB)));
        pcm_ring_barrier();
        const int b1 = buf + 1 == S ? 0 : buf + 1, bp = buf == 0 ? S - 1 : buf - 1;
        issue(bp);
        load(next, b1);
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
            for (int j = 0; j < BJ; ++j) {
                hh[i][j] = pf_mma<PF_SCALE, PF_SCALE>(cur.b[j].h, cur.a[i].h, hh[i][j]);
                qq[i][j] = pf_mma<PF_SCALE, PF_SCALE_H32>(cur.b[j].l, cur.a[i].h, qq[i][j]);
                qq[i][j] = pf_mma<PF_SCALE_H32, PF_SCALE>(cur.b[j].h, cur.a[i].l, qq[i][j]);
                qq[i][j] = pf_mma<PF_SCALE, PF_SCALE>(cur.b[j].l, cur.a[i].l, qq[i][j]);
            }
        __builtin_amdgcn_sched_barrier(0);
        buf = b1;
    };
    Frags f0, f1;
    load(f0, 0);
    int kb = 0;
    for (; kb + 1 < g.KB; kb += 2) {
        step(f0, f1);
        step(f1, f0);
    }
    if (kb < g.KB) step(f0, f1);
    __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
    __syncthreads();

    // ---- both sums into the quire, round once, store ----
    const int m_base = tm * TR + wy * 32 * BI, n_base = tn * TC + wx * 32 * BJ;
    const int half = lane >> 5;
    uint32_t any_nar = 0;
#pragma unroll
    for (int i = 0; i < BI; ++i) any_nar |= nar[wy * BI + i];
#pragma unroll
    for (int j = 0; j < BJ; ++j) any_nar |= nar[NA + wx * BJ + j];
    any_nar = __builtin_amdgcn_readfirstlane(any_nar);
    float* const badd = reinterpret_cast<float*>(lds);  // [TC]: bias * 1; the ring is free
    if (g.bias) {
        if (t < TC) {
            const uint32_t bp = tn * TC + t < g.N ? g.bias[tn * TC + t] : 0u;
            badd[t] = bp == 0x80u ? 0.0f : (float)((int32_t)Arith<P8>::stage(bp) << P8::MAXS);
            if (bp == 0x80u) atomicOr(&nar[NA + (t >> 5)], 1u << (t & 31));
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < BJ; ++j) any_nar |= __builtin_amdgcn_readfirstlane(nar[NA + wx * BJ + j]);
    }
    // The bound on HH keeps the sum below 2^31 units: it never wraps, and binary32 holds it exactly up to 2^24 units, far beyond
    // maxpos = 2^18 units, where rounding to posit<8,0> only saturates.
    auto quires = [&](int i, int j, float (&q)[16]) {
#pragma unroll
        for (int r = 0; r < 16; ++r) q[r] = __builtin_fmaf(hh[i][j][r], (float)(PF_UNIT * PF_UNIT), qq[i][j][r]);
        if (g.bias) {
#pragma unroll
            for (int r = 0; r < 16; ++r) q[r] += badd[(wx * BJ + j) * 32 + (r & 3) + 8 * (r >> 2) + 4 * half];
        }
    };
    if (g.fout != 0) {  // another output format: the sums go through LDS, and one copy of the rounding code in a loop
        uint32_t* const own = reinterpret_cast<uint32_t*>(lds) + TC + w * (BI * BJ * 1024);  // [column][row] of this wave
        static_assert((TC + W * BI * BJ * 1024) * 4 <= S * STAGE * 16, "the sums fit the ring");
#pragma unroll
        for (int j = 0; j < BJ; ++j)
#pragma unroll
            for (int i = 0; i < BI; ++i) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int c = 32 * j + (r & 3) + 8 * (r >> 2) + 4 * half;
                    own[c * (32 * BI) + 32 * i + (lane & 31)] =
                        ((uint32_t)(int32_t)hh[i][j][r] << 10) + (uint32_t)(int32_t)qq[i][j][r] + (g.bias ? (uint32_t)(int32_t)badd[wx * BJ * 32 + c] : 0u);
                }
            }
        __syncthreads();
#pragma unroll 1
        for (int e = lane; e < BI * BJ * 1024; e += 64) {
            const int c = e % (32 * BJ), r = e / (32 * BJ);
            const int m = m_base + r, n = n_base + c;
            if (m >= g.M || n >= g.N) continue;
            const bool isnar = ((nar[wy * BI + (r >> 5)] >> (r & 31)) | (nar[NA + wx * BJ + (c >> 5)] >> (c & 31))) & 1u;
            const uint32_t q1[1] = {own[c * (32 * BI) + r]};
            round_store<QuireAccum<P8>, 1>(q1, isnar, g.fout, g.C, (int64_t)m * g.ldc + n);
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
        const uint32_t cmask = nar[NA + wx * BJ + j] >> (4 * half);  // bit 8 u + b: column 8 u + 4 half + b
        const int n = n_base + 32 * j + 16 * half;
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            float q[16];
            uint32_t d[4];
            quires(i, j, q);
            const int m = m_base + 32 * i + (lane & 31);
            const bool rnar = (nar[wy * BI + i] >> (lane & 31)) & 1u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                d[u] = p8_pack4(p8_round_bits(q[4 * u]), p8_round_bits(q[4 * u + 1]), p8_round_bits(q[4 * u + 2]), p8_round_bits(q[4 * u + 3]));
                if (any_nar) {
                    const uint32_t b4 = (cmask >> (8 * u)) & 15u;
                    const uint32_t mk = rnar ? 0xFFFFFFFFu : (((b4 * 0x00204081u) & 0x01010101u) * 0xFFu);
                    d[u] = (d[u] & ~mk) | (0x80808080u & mk);
                }
            }
            // lanes l and l + 32 hold columns 8 u and 8 u + 4 of the same row: afterwards 0 .. 15 and 16 .. 31
            const auto s0 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
            const uint32_t e[4] = {s0[0], s0[1], s1[0], s1[1]};
            if (m < g.M) {
                uint8_t* c = (uint8_t*)g.C + (int64_t)m * g.ldc + n;
                if (n + 16 <= g.N) {
                    __builtin_memcpy(c, e, 16);
                } else {
#pragma unroll
                    for (int b = 0; b < 16; ++b)
                        if (n + b < g.N) c[b] = (uint8_t)(e[b >> 2] >> (8 * (b & 3)));
                }
            }
        }
    }
}

// ---- host side ----

struct P8F6Layout {
    int RBA, RBB, KB, chunks;
    int tiles_m, tiles_n;   // of 128 x 128 outputs
    size_t a_bytes, b_bytes, stat_bytes, nar_bytes, int8_bytes;
    // the int8 digits take the place of everything here where they are needed; the verdict is the last word of it
    size_t total() const { return int8_bytes; }
    bool fits() const { return a_bytes + b_bytes + nar_bytes + stat_bytes <= int8_bytes - 16; }
};

inline P8F6Layout p8_f6_layout(int64_t M, int64_t N, int64_t K) {
    P8F6Layout l;
    l.tiles_m = (int)((M + 127) / 128);
    l.tiles_n = (int)((N + 127) / 128);
    l.RBA = 4 * l.tiles_m;
    l.RBB = 4 * l.tiles_n;
    l.KB = (int)((K + 63) / 64);
    l.chunks = (l.KB + PF_CHUNK - 1) / PF_CHUNK;
    l.a_bytes = (size_t)l.KB * l.RBA * 3072;
    l.b_bytes = (size_t)l.KB * l.RBB * 3072;
    l.nar_bytes = (size_t)l.chunks * (l.tiles_m + l.tiles_n) * 16;
    l.stat_bytes = (size_t)l.chunks * (l.tiles_m + l.tiles_n) * 8;
    l.int8_bytes = p8_mfma_layout(M, N, K).total();
    return l;
}

// Products that come here, where the workspace may have up to `limit` bytes.  Timed against the int8 kernel alone on N(0, 1)
// operands (us, before -> now): 2048 x 2048 x 512 25.0 -> 24.2, x 4096 77.7 -> 57.4, 3072 x 3072 x 512 66 -> 36, 4096 x 4096 x 256
// 60 -> 35, x 4096 235 -> 153, 8192 x 512 x 2048 52 -> 45; with half the tiles the chip is half empty and the two launches
// behind weigh more: 1536^3 33.3 -> 36.4, 1024 x 2048 x 2048 34.6 -> 39.2.  Refused operands pay for the digits and a launch that
// returns (int8 kernel alone -> now, and in brackets when every tile decided for itself and the product was then taken again):
// 4096^3 N(0, 1) with one +-64 236 -> 262 (392), N(0, 8^2) 248 -> 268 (271), all patterns at random 256 -> 273 (277); one +-64 at
// 2048 x 2048 x 4096 76 -> 92 (130), 4096 x 4096 x 256 58 -> 72 (89), 8192 x 8192 x 2048 485 -> 509 (782).
inline bool p8_f6_fits(int64_t M, int64_t N, int64_t K, size_t limit) {
    return p8_mfma_fits(M, N, K) && K <= PF_MAX_K && ((M + 127) / 128) * ((N + 127) / 128) >= PF_MIN_TILES && p8_f6_layout(M, N, K).total() <= limit &&
           p8_f6_layout(M, N, K).fits();
}

inline hipError_t launch_p8_f6_gemm(hipStream_t stream, int transA, int transB, const uint8_t* A, int64_t lda, const uint8_t* B, int64_t ldb,
                                    const uint8_t* bias, void* C, int64_t ldc, int fout, int64_t M, int64_t N, int64_t K, void* workspace) {
    const P8F6Layout l = p8_f6_layout(M, N, K);
    uint8_t* base = (uint8_t*)workspace;
    uint4* Ad = reinterpret_cast<uint4*>(base);
    uint4* Bd = reinterpret_cast<uint4*>(base + l.a_bytes);
    uint32_t* nar_a = reinterpret_cast<uint32_t*>(base + l.a_bytes + l.b_bytes);
    uint32_t* nar_b = nar_a + (size_t)l.chunks * l.tiles_m * 4;
    uint2* sa = reinterpret_cast<uint2*>(base + l.a_bytes + l.b_bytes + l.nar_bytes);
    uint2* sb = sa + (size_t)l.chunks * l.tiles_m;
    uint32_t* verdict = reinterpret_cast<uint32_t*>(base + l.int8_bytes) - 1;
    // op(A)[m,k] is A[m * lda + k] unless transA; op(B)[k,n] is B[k * ldb + n] unless transB
    P8F6Job ja{A, transA ? (int64_t)1 : lda, transA ? lda : (int64_t)1, (int)M, (int)K, Ad, sa, nar_a, l.RBA, l.KB, l.chunks};
    P8F6Job jb{B, transB ? ldb : (int64_t)1, transB ? (int64_t)1 : ldb, (int)N, (int)K, Bd, sb, nar_b, l.RBB, l.KB, l.chunks};
    const unsigned blocks0 = (unsigned)l.tiles_m * (unsigned)l.chunks, blocks1 = (unsigned)l.tiles_n * (unsigned)l.chunks;
    hipLaunchKernelGGL(p8_f6_digits_kernel<0>, dim3(blocks0 + blocks1), dim3(256), 0, stream, ja, jb, blocks0, verdict);
    PNN_CHECK_LAUNCH();
    P8F6Args a{Ad, Bd, sa, sb, nar_a, nar_b, l.RBA, l.RBB, l.KB, l.chunks, bias, C, ldc, fout, (int)M, (int)N, l.tiles_m, l.tiles_n, verdict};
    hipLaunchKernelGGL(p8_f6_gemm_kernel<0>, dim3((unsigned)(l.tiles_m * l.tiles_n)), dim3(256), 0, stream, a);
    PNN_CHECK_LAUNCH();
    return launch_p8_mfma_gemm(stream, transA, transB, A, lda, B, ldb, bias, C, ldc, fout, M, N, K, base, verdict);
}

}  // namespace pnn
