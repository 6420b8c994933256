// Matrix product with the exact quire (paper Sec. 2, Sec. 3.3) on the integer matrix cores for posit(8,1), posit(8,2), the
// 10- / 12-bit formats that fit 64 bits, posit<16,1> and posit<32,2>: operands as planes of balanced base-256 digits
// (dig_planes.h).
//
// Launches of a call: a scan of both operands (which window of digits serves), the digit planes of both, then one product
// kernel per plane count, of which the one that was decided on does the work and the others return at once, and the
// merge of a reduction cut into slices.
//
// Layout of the rewritten operands: [k block of 32][row block of 32][plane][lane][16 bytes] in the lane order of
// v_mfma_i32_32x32x32_i8 (gemm_p8_mfma.h), and one byte per (k block, row block): bit g is set when group g of the planes
// (DigGroups) holds a non-zero digit in the block.
#pragma once

#include "dig_planes.h"

namespace pnn {

struct DigMatrixJob {
    const void* src;
    int64_t s_r, s_k;   // element (row, k) at src[row * s_r + k * s_k]; one of the two is 1
    int rows, K;
    uint8_t* mask;      // [KB][RB]: which groups of planes of the block hold anything
    int RB;
};

constexpr int DIG_ROWS = 128;  // rows of a workgroup of the digit launch: four row blocks, one wave each

// Planes of one k block and four row blocks.  An operand stored reduction-index-major goes through an LDS tile.
template <class F, int NP>
__device__ __forceinline__ void dig_matrix_planes(const DigMatrixJob& job, uint8_t* __restrict__ dst, int base, int kb, int bx,
                                                  const typename Storage<F::N>::T (*tile)[DIG_ROWS], uint64_t* tab) {
    typedef typename Storage<F::N>::T T;
    typedef typename DigWord<NP>::T W;
    constexpr int V = 16 / (int)sizeof(T);
    const int t = threadIdx.x;
    const bool via_lds = job.s_k != 1;
    if constexpr (F::N == 8) {
        tab[t] = dig_word<F, NP>((uint32_t)t, base);
        __syncthreads();
    }
    const int rb = bx * 4 + (t >> 6), lane = t & 63;  // a wave: one row block
    if (rb >= job.RB) return;
    const int row = rb * 32 + (lane & 31), k0 = kb * 32 + 16 * (lane >> 5);
    uint32_t pat[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) pat[b] = 0;
    if (via_lds) {
#pragma unroll
        for (int b = 0; b < 16; ++b) pat[b] = tile[16 * (lane >> 5) + b][(t >> 6) * 32 + (lane & 31)];
    } else if (row < job.rows) {
        const T* p = (const T*)job.src + (int64_t)row * job.s_r + k0;
        if (k0 + 16 <= job.K && (((uintptr_t)p) & 15u) == 0) {
#pragma unroll
            for (int c = 0; c < 16 / V; ++c) {
                const uint4 v = reinterpret_cast<const uint4*>(p)[c];
                const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int b = 0; b < V; ++b)
                    pat[c * V + b] = sizeof(T) == 4 ? wv[b & 3] : (wv[b * (int)sizeof(T) / 4] >> (8 * ((b * (int)sizeof(T)) & 3))) & (sizeof(T) == 1 ? 0xFFu : 0xFFFFu);
            }
        } else {
#pragma unroll
            for (int b = 0; b < 16; ++b)
                if (k0 + b < job.K) pat[b] = p[b];
        }
    }
    W w[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) {
        if constexpr (F::N == 8) w[b] = (W)tab[pat[b]];
        else w[b] = dig_word<F, NP>(pat[b] & F::MASK, base);
    }
    uint32_t pl[NP][4];
    dig_planes_of<NP>(w, pl);
    uint4* out = reinterpret_cast<uint4*>(dst) + ((int64_t)(kb * job.RB + rb) * NP) * 64 + lane;
    uint32_t mask = 0;
#pragma unroll
    for (int g = 0; g < DigGroups<NP>::G; ++g) {
        uint32_t any = 0;
#pragma unroll
        for (int i = DigGroups<NP>::start(g); i < DigGroups<NP>::start(g + 1); ++i) any |= pl[i][0] | pl[i][1] | pl[i][2] | pl[i][3];
        if (__ballot(any != 0) != 0) mask |= 1u << g;
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) out[i * 64] = make_uint4(pl[i][0], pl[i][1], pl[i][2], pl[i][3]);
    if (lane == 0) job.mask[(int64_t)kb * job.RB + rb] = (uint8_t)mask;
}

// Both operands in one launch: the first blocks0 workgroups take job0, the rest job1.  planes: where the planes of A start;
// those of B follow at the place the decided plane count gives.
template <class F>
__global__ __launch_bounds__(256) void dig_matrix_kernel(DigMatrixJob job0, DigMatrixJob job1, unsigned blocks0, const void* __restrict__ stats,
                                                         DigInfo* __restrict__ info, uint8_t* __restrict__ planes, int KB, int narrow) {
    typedef typename Storage<F::N>::T T;
    typedef DigFormat<F> D;
    __shared__ __attribute__((aligned(16))) T tile[32][DIG_ROWS];
    __shared__ uint64_t tab[F::N == 8 ? 256 : 1];
    const bool first = blockIdx.x < blocks0;
    const DigMatrixJob& job = first ? job0 : job1;
    const unsigned lin = first ? blockIdx.x : blockIdx.x - blocks0;
    const unsigned gx = (unsigned)((job.RB + 3) / 4);
    const int bx = (int)(lin % gx), kb = (int)(lin / gx);
    const int t = threadIdx.x;
    if (job.s_k != 1) {
        constexpr int V = 16 / (int)sizeof(T), W = 16 / V;  // thread: 16 consecutive rows at one k, in W words of 16 bytes
        const int kk = t >> 3, seg = (t & 7) * 16;
        const int k = kb * 32 + kk;
        const int row0 = bx * DIG_ROWS + seg;
        const T* p = (const T*)job.src + (int64_t)k * job.s_k + row0;
        T* dt = &tile[kk][seg];
        if (k < job.K && row0 + 16 <= job.rows && (((uintptr_t)p) & 15u) == 0) {
            uint4 v[W];
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = reinterpret_cast<const uint4*>(p)[c];
#pragma unroll
            for (int c = 0; c < W; ++c) reinterpret_cast<uint4*>(dt)[c] = v[c];
        } else {
            T v[16];
#pragma unroll
            for (int b = 0; b < 16; ++b) v[b] = (k < job.K && row0 + b < job.rows) ? p[b] : (T)0;
#pragma unroll
            for (int b = 0; b < 16; ++b) dt[b] = v[b];
        }
    }
    const DigInfo d = dig_read_decision<F, dig_stat_packed<F>()>(stats, info, narrow != 0, blockIdx.x == 0);
    if (d.np == 0) return;
    __syncthreads();
    uint8_t* dst = first ? planes : planes + (int64_t)KB * job0.RB * d.np * 1024;
    const int base = first ? d.base[0] : d.base[1];
    if (D::NP1 != 0 && d.np == D::NP1) dig_matrix_planes<F, (D::NP1 ? D::NP1 : D::NP2)>(job, dst, base, kb, bx, tile, tab);
    else dig_matrix_planes<F, D::NP2>(job, dst, base, kb, bx, tile, tab);
}

struct DigGemmArgs {
    uint8_t* planes;              // A's planes, B's behind them
    const uint8_t* ma;
    const uint8_t* mb;
    const DigInfo* info;
    int RBA, RBB, KB;
    int splits, kb_per_split;     // slices of the reduction (gridDim.y)
    uint32_t* part;               // [slice][limb][M N], null without slices; flags behind them
    uint32_t* rowflag;            // [slice][M]
    uint32_t* colflag;            // [slice][N]
    const void* bias;
    void* C;
    int64_t ldc;
    FmtRT fin, fout;
    int M, N, tiles_m, tiles_n;
};


// Rounds and stores rows first, first + STEP, ... of one column, four in flight.
template <int L, class T, int STEP, class Value, class IsNar>
__device__ __forceinline__ void dig_store_rows(int first, int rows, const DigRound& d, T* dst, int64_t ld, const Value& value, const IsNar& is_nar) {
    const int qfrac = d.qfrac();
#pragma unroll 1
    for (int lr0 = first; lr0 < rows; lr0 += 4 * STEP) {
        uint32_t res[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int lr = lr0 + u * STEP < 64 ? lr0 + u * STEP : 63;
            uint32_t q[L];
            value(lr, q);
            const uint32_t v = dig_round_limbs<L, sizeof(T) == 4>(q, qfrac, d.fout);
            res[u] = is_nar(lr) ? d.fout.nar() : v;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (lr0 + u * STEP < rows) dst[(int64_t)(lr0 + u * STEP) * ld] = (T)res[u];
    }
}

// Rounds and stores rows first, first + STEP, ... of column n of a tile that starts at row row0, the bias added where there is one.
// value(row, limbs) gives the integer of the sums in units of minpos^2 2^at; cnar, row_flag(row): whether column or row meet NaR.
template <int L, int STEP, class Value, class Flag>
__device__ __forceinline__ void dig_round_column(const DigGemmArgs& g, int at, int row0, int n, int first, int rows, uint32_t cnar, const Value& value,
                                                 const Flag& row_flag) {
    DigRound rd;
    rd.fin = g.fin;
    rd.fout = g.fout;
    rd.at = at;
    auto is_nar = [&](int lr) { return (cnar | row_flag(lr)) != 0; };
    auto store = [&](auto limbs, const auto& of) {
        constexpr int W = limbs;
        const int64_t base = (int64_t)row0 * g.ldc + n;
        if (rd.fout.n <= 8) dig_store_rows<W, uint8_t, STEP>(first, rows, rd, (uint8_t*)g.C + base, g.ldc, of, is_nar);
        else if (rd.fout.n <= 16) dig_store_rows<W, uint16_t, STEP>(first, rows, rd, (uint16_t*)g.C + base, g.ldc, of, is_nar);
        else dig_store_rows<W, uint32_t, STEP>(first, rows, rd, (uint32_t*)g.C + base, g.ldc, of, is_nar);
    };
    if (g.bias) {
        // The bias is decoded once per column, and the rows go four at a time as without it (decoded at every row, one row at
        // a time: 784 x 2976 x 631 posit(8,1) 50 us, now 44).  A value is a multiple of 2^maxs minpos^2, so where the sums'
        // unit is no larger and the bias fits their limbs it is added in that unit; else both are placed in 128 bits (46).
        const uint32_t bp = dig_load_pattern(g.bias, n, rd.fin.n);
        const __int128 bias = dig_bias_value(bp, rd.fin);
        cnar |= bp == rd.fin.nar() ? 1u : 0u;
        const int maxs = rd.fin.maxs();
        if (L <= 4 && at <= maxs && 3 * maxs - at <= 32 * L - 3) {
            const __int128 placed = at >= 0 ? bias >> at : (__int128)((unsigned __int128)bias << -at);
            uint32_t bl[L];
#pragma unroll
            for (int l = 0; l < L; ++l) bl[l] = (uint32_t)(placed >> (l < 4 ? 32 * l : 127));
            auto biased = [&](int lr, uint32_t (&u)[L]) {
                uint32_t b[L];
                value(lr, u);
#pragma unroll
                for (int l = 0; l < L; ++l) b[l] = bl[l];
                quire_merge<L>(u, b);
            };
            store(dig_int<L>(), biased);
            return;
        }
        auto biased = [&](int lr, uint32_t (&u)[4]) {
            uint32_t q[L];
            value(lr, q);
            dig_add_bias<L>(q, at, bias, u);
        };
        rd.at = 0;
        store(dig_int<4>(), biased);
    } else {
        store(dig_int<L>(), value);
    }
}

// 64 x 64 outputs per workgroup: KG groups of four waves (2 x 2), a wave owns one block of 32 x 32 and its 2 NP - 1 sums
// over the k blocks of its group (every KG-th).  The runs of a k block go straight into LDS, a ring of S blocks with copies
// S - 1 blocks ahead.  The waves of a workgroup leave each barrier together and would all wait for their LDS reads
// together, so the operand registers of a step are read during the step before (two sets).  What a step costs beside its
// matrix instructions is scalar code, hence the straight-line loop over a fixed set of planes (DigGroups).  Registers decide
// how many waves a SIMD holds: 5 sums three, 7 sums two; more planes go to dig_gemm_pair_kernel.
template <int NP, int KG, int S>
__global__ __launch_bounds__(256 * KG, (NP <= 3 ? 3 : 2)) void dig_gemm_kernel(DigGemmArgs g) {
    static_assert(NP == 3 || NP == 4, "planes whose sums leave room for two waves on a SIMD");
    typedef DigGroups<NP> D;
    constexpr int NC = 2 * NP - 1, L = dig_limbs<NP>();
    constexpr int RPB = 4 * NP;  // runs of 1 KB per k block: two row blocks and two column blocks of NP planes
    constexpr int MAXKB = DIG_MAXK / 32 + 1;
    if (__builtin_amdgcn_readfirstlane(g.info->np) != NP) return;
    // One LDS object: beside a second one the compiler tells the objects apart and puts a wait for EVERY outstanding copy in
    // front of each read of the ring (1024^3 posit<16,1>: 1.2 us a step).
    constexpr int RING = KG * S * RPB * 64, MASKW = (4 * MAXKB + 15) / 16;  // words of 16 bytes
    constexpr int LISTW = (2 * MAXKB + 15) / 16;
    __shared__ uint4 lds[RING + MASKW + KG * 32 + 1 + LISTW];
    uint4* const stage = lds;                                          // [KG * S][RPB * 64]
    uint8_t* const masks = reinterpret_cast<uint8_t*>(lds + RING);     // [4][MAXKB]: the tile's row blocks 0, 1 and column blocks 0, 1 over the slice
    uint32_t* const rowv = reinterpret_cast<uint32_t*>(lds + RING + MASKW);  // [KG][64]
    uint32_t* const colv = rowv + KG * 64;
    uint32_t* const present = colv + KG * 64;                          // k blocks that hold anything in groups 0 and 1; entries of the list
    uint16_t* const list = reinterpret_cast<uint16_t*>(present + 4);   // k blocks that hold anything below the main loop's planes
    static_assert(KG * L * 64 * 64 * 4 <= RING * 16, "the outputs' integers pass through the ring");

    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int w = wave & 3, kg = wave >> 2;
    const int wy = w >> 1, wx = w & 1;
    // XCD-aware order, as in gemm_p8_mfma.h: each XCD a contiguous run of tiles, walked in bands of 8 tile-rows
    const int nblk = g.tiles_m * g.tiles_n;
    int lid = blockIdx.x;
    if ((nblk & 7) == 0) lid = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
    const int band = lid / (8 * g.tiles_n);
    const int band_rows = (g.tiles_m - band * 8) < 8 ? (g.tiles_m - band * 8) : 8;
    const int in_band = lid - band * 8 * g.tiles_n;
    const int tm = band * 8 + in_band % band_rows, tn = in_band / band_rows;
    const int z = blockIdx.y;
    const int kb0 = z * g.kb_per_split;
    const int nkb = (kb0 + g.kb_per_split < g.KB ? kb0 + g.kb_per_split : g.KB) - kb0;
    const int nst = (nkb + KG - 1) / KG;  // steps of the workgroup; group kg multiplies k blocks kb0 + step * KG + kg

    // wave w of a group copies block w of the k block's four (A: row block 0, 1; B: column block 0, 1)
    const int64_t rbx = (w < 2) ? g.RBA : g.RBB;
    const int blk = (w < 2) ? tm * 2 + w : tn * 2 + (w - 2);
    const uint4* const src0 = reinterpret_cast<const uint4*>(g.planes) + ((w < 2) ? 0 : (int64_t)g.KB * g.RBA * NP * 64) + (kb0 * rbx + blk) * (NP * 64) + lane;
    const int64_t adv = rbx * (KG * NP * 64);
    const uint4* src = src0 + kg * rbx * (NP * 64);
    auto copy = [&](auto sp, const uint4* from, uint4* to) {
#pragma unroll
        for (int c = sp; c < NP; ++c)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(from + c * 64),
                                             (__attribute__((address_space(3))) void*)(to + c * 64), 16, 0, 0);
    };
    uint4* const ring = stage + kg * S * (RPB * 64) + w * NP * 64;  // where this wave's block of buffer 0 goes
    // The first S - 1 blocks are copied whole while the masks come in.
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        if (s * KG + kg < nkb) copy(dig_int<0>(), src, ring + s * (RPB * 64));
        src += adv;
    }
    if (t < 3) present[t] = 0;
    const int a_nar = __builtin_amdgcn_readfirstlane(g.info->nar[0]), b_nar = __builtin_amdgcn_readfirstlane(g.info->nar[1]);
    const int at = __builtin_amdgcn_readfirstlane(g.info->base[0] + g.info->base[1]);
    __syncthreads();
    for (int k = t; k < nkb; k += 256 * KG) {
        uint32_t any = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t m = b < 2 ? g.ma[(int64_t)(kb0 + k) * g.RBA + tm * 2 + b] : g.mb[(int64_t)(kb0 + k) * g.RBB + tn * 2 + (b - 2)];
            masks[b * MAXKB + k] = (uint8_t)m;
            any |= m;
        }
        if (any & 1u) atomicAdd(&present[0], 1u);
        if (any & 2u) atomicAdd(&present[1], 1u);
    }
    __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));  // block 0 is read behind the barrier, ahead of the first step
    __syncthreads();
    // The straight-line loop starts at the first group that more than a quarter of the k blocks use: below that the second
    // look at those blocks is cheaper than multiplying the group everywhere.
    const uint32_t p0 = __builtin_amdgcn_readfirstlane(present[0]), p1 = __builtin_amdgcn_readfirstlane(present[1]);
    const int g0 = 4 * p0 > (uint32_t)nkb ? 0 : 4 * p1 > (uint32_t)nkb ? 1 : 2;
    const uint32_t below = (1u << g0) - 1u;
    for (int k = t; k < nkb; k += 256 * KG)
        if ((masks[k] | masks[MAXKB + k] | masks[2 * MAXKB + k] | masks[3 * MAXKB + k]) & below) list[atomicAdd(&present[2], 1u)] = (uint16_t)k;

    pm_v16i acc[NC];
#pragma unroll
    for (int s = 0; s < NC; ++s)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[s][r] = 0;
    uint32_t row_nar = 0, col_nar = 0;
    const uint4* const sa0 = stage + kg * S * (RPB * 64) + wy * NP * 64 + lane;
    const uint4* const sb0 = stage + kg * S * (RPB * 64) + (2 + wx) * NP * 64 + lane;
    DigFrag<NP> f0, f1;
    auto loop = [&](auto sp) {
        constexpr int SP = sp;
        // One step: block st is in cur.  Before the barrier this wave's copies of block st + 1 have landed; behind it
        // everyone's have, and everyone's reads of block st - 1 (issued in step st - 2) have been consumed, so its buffer
        // takes a copy.  Copies complete in order; near the end fewer are in flight, so all are waited for.
        auto step = [&](int st, const DigFrag<NP>& cur, DigFrag<NP>& next) {
            const int kb = st * KG + kg, kn = kb + (S - 1) * KG;
            if (st > 0 && kb + (S - 2) * KG < nkb) __builtin_amdgcn_s_waitcnt(pcm_vmcnt((S - 3) * (NP - SP)));
            else __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
            pcm_ring_barrier();
            if (kn < nkb) {
                copy(sp, src, ring + ((st + S - 1) % S) * (RPB * 64));
                src += adv;
            }
            const int nb = ((st + 1) % S) * (RPB * 64);
            next.template load<SP>(sa0 + nb, sb0 + nb);  // beyond the last block: whatever the buffer holds, not used
            if (kb < nkb) {
                if (a_nar) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) row_nar |= pm_marker_bits((uint32_t)cur.a[NP - 1][i]);
                }
                if (b_nar) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) col_nar |= pm_marker_bits((uint32_t)cur.b[NP - 1][i]);
                }
                dig_mma<NP, SP, NP, SP, NP>(cur, acc);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        f0.template load<SP>(sa0, sb0);
        for (int st = 0; st < nst; st += 2) {
            step(st, f0, f1);
            if (st + 1 < nst) step(st + 1, f1, f0);
        }
    };
    if (g0 == 0) loop(dig_int<0>());
    else if (g0 == 1) loop(dig_int<D::start(1)>());
    else loop(dig_int<D::start(2)>());
    __syncthreads();
    // The k blocks with anything below: the first group's waves copy and multiply them once more, the pairs left out only;
    // S at a time, so that their copies' latencies overlap.
    const int extra = __builtin_amdgcn_readfirstlane((int)present[2]);
    for (int e0 = 0; e0 < extra; e0 += S) {
        const int ne = extra - e0 < S ? extra - e0 : S;
        if (kg == 0)
            for (int e = 0; e < ne; ++e) copy(dig_int<0>(), src0 + __builtin_amdgcn_readfirstlane((int)list[e0 + e]) * rbx * (NP * 64), ring + e * (RPB * 64));
        __builtin_amdgcn_s_waitcnt(pcm_vmcnt(0));
        __syncthreads();
        if (kg == 0) {
#pragma unroll 1
            for (int e = 0; e < ne; ++e) {
                const int k = list[e0 + e];
                f0.template load<0>(sa0 + e * (RPB * 64), sb0 + e * (RPB * 64));
                dig_mma_below<NP, 0, 0>(g0, __builtin_amdgcn_readfirstlane((uint32_t)masks[wy * MAXKB + k]),
                                        __builtin_amdgcn_readfirstlane((uint32_t)masks[(2 + wx) * MAXKB + k]), f0, acc);
            }
        }
        __syncthreads();
    }

    // ---- NaR flags, and the sums as one integer per output, to LDS; then rounded and stored (or left for the merge) along
    // the rows: the matrix instruction leaves a lane with 16 rows of one column, and one copy of the rounding code in a loop
    // costs fewer instruction fetches than sixteen ----
    uint32_t* vals = reinterpret_cast<uint32_t*>(stage) + kg * (L * 4096);
    row_nar = (row_nar | (uint32_t)__shfl_xor((int)row_nar, 32)) & 0x80808080u;
    col_nar = (col_nar | (uint32_t)__shfl_xor((int)col_nar, 32)) & 0x80808080u;
    if (lane < 32) {
        if (wx == 0) rowv[kg * 64 + wy * 32 + lane] = row_nar;  // the two waves of a row block saw the same rows
        if (wy == 0) colv[kg * 64 + wx * 32 + lane] = col_nar;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int lr = wy * 32 + (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5);
        uint32_t q[L];
        dig_combine<NP>(acc, r, q);
#pragma unroll
        for (int l = 0; l < L; ++l) vals[l * 4096 + lr * 64 + wx * 32 + (lane & 31)] = q[l];
    }
    __syncthreads();
    const uint32_t* const all = reinterpret_cast<const uint32_t*>(stage);
    const bool sliced = gridDim.y > 1;
    const int n = tn * 64 + lane;
    uint32_t cnar = colv[lane];
    if (KG == 2) cnar |= colv[(KG - 1) * 64 + lane];
    if (sliced) {
        // the first tile column stores the row flags of its tile row, the first tile row the column flags: all of them
        if (tn == 0 && t < 64 && tm * 64 + t < g.M) g.rowflag[(int64_t)z * g.M + tm * 64 + t] = rowv[t] | (KG == 2 ? rowv[(KG - 1) * 64 + t] : 0u);
        if (tm == 0 && t < 64 && n < g.N) g.colflag[(int64_t)z * g.N + n] = cnar;
    }
    if (n >= g.N) return;
    auto value = [&](int lr, uint32_t (&q)[L]) {
#pragma unroll
        for (int l = 0; l < L; ++l) q[l] = all[l * 4096 + lr * 64 + lane];
        if (KG == 2) {
            uint32_t o[L];
#pragma unroll
            for (int l = 0; l < L; ++l) o[l] = all[(KG - 1) * (L * 4096) + l * 4096 + lr * 64 + lane];
            quire_merge<L>(q, o);
        }
    };
    const int rows = g.M - tm * 64 < 64 ? g.M - tm * 64 : 64;
    if (sliced) {
        const int64_t MN = (int64_t)g.M * g.N;
#pragma unroll 2
        for (int lr = wave; lr < rows; lr += 4 * KG) {
            uint32_t q[L];
            value(lr, q);
#pragma unroll
            for (int l = 0; l < L; ++l) g.part[((int64_t)z * L + l) * MN + (int64_t)(tm * 64 + lr) * g.N + n] = q[l];
        }
        return;
    }
    dig_round_column<L, 4 * KG>(g, at, tm * 64, n, wave, rows, cnar, value, [&](int lr) { return rowv[lr] | (KG == 2 ? rowv[(KG - 1) * 64 + lr] : 0u); });
}

// 64 x 32 outputs per workgroup, a wave 16 x 32 of them, whose 2 NP - 1 sums (120 registers for eight planes, 56 for four) leave room for a second
// workgroup on the CU, four with four planes.  LDS holds one pair of k blocks; its operands go to registers before the next pair's copies start, and the
// other workgroups multiply meanwhile.  Blocks of 32 x 32 outputs per wave left one wave to a SIMD with eight planes, which waited for every barrier, LDS read
// and rounding alone.  us a call, 1 % of extremes, 32 x 32 -> now: posit<16,1> 1024^3 65.5 and 58.7, 971 x 1044 x 976 111 and 81, 4096^3 2697 and 2145,
// posit(8,2) 512 x 512 x 8192 274 and 172; posit<32,2>, N(0, 1), 1024^3 52.7 and 47.5.
// MANY: tiles in two dimensions of the launch.
template <int NP, bool MANY>
__global__ __launch_bounds__(256, (NP <= 4 ? 4 : 2)) void dig_gemm_pair_kernel(DigGemmArgs g) {
    typedef DigGroups<NP> D;
    constexpr int NC = 2 * NP - 1, L = dig_limbs<NP>(), TR = 64, TC = 32;
    constexpr int RPB = 3 * NP;  // runs of 1 KB per k block: two row blocks and a column block of NP planes
    constexpr int MAXP = (DIG_MAXK / 32 + 2) / 2;
    if (__builtin_amdgcn_readfirstlane(g.info->np) != NP) return;
    // one LDS object (see dig_gemm_kernel)
    constexpr int VALS = L * TR * TC / 4, RING = 2 * RPB * 64 > VALS ? 2 * RPB * 64 : VALS;  // words of 16 bytes
    constexpr int MASKW = (3 * MAXP + 15) / 16, LISTW = (2 * MAXP + 15) / 16;
    __shared__ uint4 lds[RING + MASKW + (TR + TC) / 4 + 1 + LISTW];
    uint4* const stage = lds;
    uint8_t* const masks = reinterpret_cast<uint8_t*>(lds + RING);     // [3][MAXP]: the tile's row blocks 0, 1 and its column block, by pairs
    uint32_t* const rowv = reinterpret_cast<uint32_t*>(lds + RING + MASKW);
    uint32_t* const colv = rowv + TR;
    uint32_t* const present = colv + TC;                               // pairs that hold anything in groups 0 and 1; entries of the list
    uint16_t* const list = reinterpret_cast<uint16_t*>(present + 4);   // pairs that hold anything below the main loop's planes

    const int t = threadIdx.x;
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    // XCD-aware order, as in gemm_p8_mfma.h: each XCD a contiguous run of tiles, walked in bands of 8 tile-rows
    const int nblk = g.tiles_m * g.tiles_n;
    int lid = MANY ? dig_tile_id() : (int)blockIdx.x;
    if (MANY && lid >= nblk) return;
    if ((nblk & 7) == 0) lid = (lid & 7) * (nblk >> 3) + (lid >> 3);
    const int band = lid / (8 * g.tiles_n);
    const int band_rows = (g.tiles_m - band * 8) < 8 ? (g.tiles_m - band * 8) : 8;
    const int in_band = lid - band * 8 * g.tiles_n;
    const int tm = band * 8 + in_band % band_rows, tn = in_band / band_rows;
    const int z = blockIdx.y;
    const int kb0 = z * g.kb_per_split;
    const int nkb = (kb0 + g.kb_per_split < g.KB ? kb0 + g.kb_per_split : g.KB) - kb0;
    const int whole = nkb / 2;  // pairs; an odd block behind them is multiplied in all its planes

    const uint4* const pa = reinterpret_cast<const uint4*>(g.planes) + ((int64_t)kb0 * g.RBA + tm * 2) * (NP * 64) + lane;
    const uint4* const pb = reinterpret_cast<const uint4*>(g.planes) + ((int64_t)g.KB * g.RBA + (int64_t)kb0 * g.RBB + tn) * (NP * 64) + lane;
    // wave w copies planes SP + w, SP + w + 4 of the three blocks
    typedef __attribute__((address_space(3))) uint4 LdsQuad;
    LdsQuad* const ring = (LdsQuad*)lds;
    auto issue = [&](auto sp, int p) {
        constexpr int SP = sp;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = 2 * p + h;
            if (k >= nkb) break;
            const uint4* const ka = pa + (int64_t)k * g.RBA * (NP * 64);
            const uint4* const kb = pb + (int64_t)k * g.RBB * (NP * 64);
#pragma unroll
            for (int i = 0; i < (NP - SP + 3) / 4; ++i) {
                const int c = SP + w + 4 * i;
                if (c >= NP) continue;
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(b < 2 ? ka + (b * NP + c) * 64 : kb + c * 64),
                                                     (__attribute__((address_space(3))) void*)(ring + (h * RPB + b * NP + c) * 64), 16, 0, 0);
            }
        }
    };
    issue(dig_int<0>(), 0);
    if (t < 3) present[t] = 0;
    const int a_nar = __builtin_amdgcn_readfirstlane(g.info->nar[0]), b_nar = __builtin_amdgcn_readfirstlane(g.info->nar[1]);
    const int at = __builtin_amdgcn_readfirstlane(g.info->base[0] + g.info->base[1]);
    __syncthreads();
    for (int p = t; p < whole; p += 256) {
        uint32_t any = 0;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            uint32_t m = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t k = kb0 + 2 * p + h;
                m |= b < 2 ? g.ma[k * g.RBA + tm * 2 + b] : g.mb[k * g.RBB + tn];
            }
            masks[b * MAXP + p] = (uint8_t)m;
            any |= m;
        }
        if (any & 1u) atomicAdd(&present[0], 1u);
        if (any & 2u) atomicAdd(&present[1], 1u);
    }
    __syncthreads();
    // The straight-line loop starts at the first group that more than a quarter of the pairs use (see dig_gemm_kernel); of five and six planes half of them
    // (1024^3, N(0, 1) with extremes, (10,1) 41.5 and 38.6 us, (12,1) 48.0 and 47.2; posit(8,2) with four planes, 4096 x 4096 x 1024, 155 and 171; posit<32,2> 4096^3 1667 and 2252).
    constexpr uint32_t SHARE = NP == 5 || NP == 6 ? 2 : 4;
    const uint32_t p0 = __builtin_amdgcn_readfirstlane(present[0]), p1 = __builtin_amdgcn_readfirstlane(present[1]);
    const int g0 = SHARE * p0 > (uint32_t)whole ? 0 : SHARE * p1 > (uint32_t)whole ? 1 : 2;
    const uint32_t below = (1u << g0) - 1u;
    for (int p = t; p < whole; p += 256)
        if ((masks[p] | masks[MAXP + p] | masks[2 * MAXP + p]) & below) list[atomicAdd(&present[2], 1u)] = (uint16_t)p;

    dig_v4i acc[2][NC];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < NC; ++s) acc[h][s] = dig_v4i{0, 0, 0, 0};
    uint32_t row_nar = 0, col_nar[2] = {0, 0};
    const uint4* const lane0 = stage + (lane >> 5) * (RPB * 64) + ((lane >> 4) & 1) * 32 + (lane & 15);
    const uint4* const sa0 = lane0 + (w >> 1) * NP * 64 + (w & 1) * 16;
    const uint4* const sb0 = lane0 + 2 * NP * 64;
    // This wave's copies are in LDS; behind the barrier everyone's are.
    auto landed = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0), lgkmcnt(0)
        pcm_ring_barrier();
    };
    // Everyone has read the pair: LDS takes the next one.
    auto taken = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        pcm_ring_barrier();
    };
    auto loop = [&](auto sp) {
        constexpr int SP = sp;
#pragma unroll 1
        for (int p = 0; p < whole; ++p) {
            DigPair<NP> f;
            landed();
            f.template load<SP>(sa0, sb0);
            if (p + 1 < whole) {
                taken();
                issue(sp, p + 1);
            } else if (nkb & 1) {
                taken();
                issue(dig_int<0>(), p + 1);
            }
            dig_pair_markers<NP>(a_nar, b_nar, f, row_nar, col_nar);
            dig_pair_mma<NP, SP, NP, SP, NP>(f, acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (g0 == 0) loop(dig_int<0>());
    else if (g0 == 1) loop(dig_int<D::start(1)>());
    else loop(dig_int<D::start(2)>());
    if (nkb & 1) {
        landed();
        const int to = -(lane >> 5) * (RPB * 64);
        dig_single_mma<NP>(sa0 + to, sb0 + to, lane, a_nar, b_nar, row_nar, col_nar, acc);
    }
    __syncthreads();
    // the pairs with anything below once more, the planes left out only
    const int extra = __builtin_amdgcn_readfirstlane((int)present[2]);
    if (extra > 0) issue(dig_int<0>(), __builtin_amdgcn_readfirstlane((int)list[0]));
#pragma unroll 1
    for (int e = 0; e < extra; ++e) {
        const int p = list[e];
        const uint32_t ma = __builtin_amdgcn_readfirstlane((uint32_t)masks[(w >> 1) * MAXP + p]), mb = __builtin_amdgcn_readfirstlane((uint32_t)masks[2 * MAXP + p]);
        DigPair<NP> f;
        landed();
        f.template load<0>(sa0, sb0);
        if (e + 1 < extra) {
            const int next = __builtin_amdgcn_readfirstlane((int)list[e + 1]);
            taken();
            issue(dig_int<0>(), next);
        }
        dig_pair_below<NP, 0, 0>(g0, ma, mb, f, acc);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();

    // ---- NaR flags, and the sums as one integer per output, to LDS; then rounded and stored (or left for the merge) ----
    uint32_t* const vals = reinterpret_cast<uint32_t*>(stage);
    row_nar = dig_pair_across(row_nar);
#pragma unroll
    for (int h = 0; h < 2; ++h) col_nar[h] = dig_pair_across(col_nar[h]);
    if (lane < 16) {
        rowv[w * 16 + lane] = row_nar;
        if (w == 0) {  // the four waves saw the same columns
#pragma unroll
            for (int h = 0; h < 2; ++h) colv[16 * h + lane] = col_nar[h];
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int lr = w * 16 + 4 * (lane >> 4) + r;
            uint32_t q[L];
            dig_combine<NP>(acc[h], r, q);
#pragma unroll
            for (int l = 0; l < L; ++l) vals[l * (TR * TC) + lr * TC + 16 * h + (lane & 15)] = q[l];
        }
    __syncthreads();
    constexpr int STEP = 256 / TC;
    const bool sliced = gridDim.y > 1;
    const int col = t % TC, first = t / TC, n = tn * TC + col;
    const uint32_t cnar = colv[col];
    if (sliced) {
        // the first tile column stores the row flags of its tile row, the first tile row the column flags: all of them
        if (tn == 0 && t < TR && tm * TR + t < g.M) g.rowflag[(int64_t)z * g.M + tm * TR + t] = rowv[t];
        if (tm == 0 && t < TC && n < g.N) g.colflag[(int64_t)z * g.N + n] = cnar;
    }
    if (n >= g.N) return;
    auto value = [&](int lr, uint32_t (&q)[L]) {
#pragma unroll
        for (int l = 0; l < L; ++l) q[l] = vals[l * (TR * TC) + lr * TC + col];
    };
    const int rows = g.M - tm * TR < TR ? g.M - tm * TR : TR;
    if (sliced) {
        const int64_t MN = (int64_t)g.M * g.N;
#pragma unroll 2
        for (int lr = first; lr < rows; lr += STEP) {
            uint32_t q[L];
            value(lr, q);
#pragma unroll
            for (int l = 0; l < L; ++l) g.part[((int64_t)z * L + l) * MN + (int64_t)(tm * TR + lr) * g.N + n] = q[l];
        }
        return;
    }
    dig_round_column<L, STEP>(g, at, tm * TR, n, first, rows, cnar, value, [&](int lr) { return rowv[lr]; });
}

// Products of few tiles: 32 x 32 outputs per workgroup, whose KG waves share the reduction (wave kg the k blocks kg, kg + KG, ...).
// No wave shares an operand with another, so the blocks go from memory straight to registers, two ahead, without LDS or a
// barrier until the sums meet.  With 64 x 64 tiles such a product has a fraction of the chip's workgroups, each bound by its own
// latency: the fill of the ring, a few steps, 16 outputs rounded per thread instead of four.
template <int NP, int KG>
__global__ __launch_bounds__(64 * KG, 2) void dig_gemm_small_kernel(DigGemmArgs g) {
    constexpr int NC = 2 * NP - 1, L = dig_limbs<NP>();
    if (__builtin_amdgcn_readfirstlane(g.info->np) != NP) return;
    __shared__ uint32_t lds[KG * (L * 1024 + 64)];
    const int t = threadIdx.x;
    const int lane = t & 63, kg = __builtin_amdgcn_readfirstlane(t >> 6);
    const int tm = blockIdx.x % g.tiles_m, tn = blockIdx.x / g.tiles_m;
    const int a_nar = __builtin_amdgcn_readfirstlane(g.info->nar[0]), b_nar = __builtin_amdgcn_readfirstlane(g.info->nar[1]);
    const int at = __builtin_amdgcn_readfirstlane(g.info->base[0] + g.info->base[1]);
    const uint4* sa = reinterpret_cast<const uint4*>(g.planes) + ((int64_t)kg * g.RBA + tm) * (NP * 64) + lane;
    const uint4* sb = reinterpret_cast<const uint4*>(g.planes) + ((int64_t)g.KB * g.RBA + (int64_t)kg * g.RBB + tn) * (NP * 64) + lane;
    const int64_t a_adv = (int64_t)KG * g.RBA * (NP * 64), b_adv = (int64_t)KG * g.RBB * (NP * 64);
    pm_v16i acc[NC];
#pragma unroll
    for (int s = 0; s < NC; ++s)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[s][r] = 0;
    uint32_t row_nar = 0, col_nar = 0;
    const int n_steps = g.KB > kg ? (g.KB - kg + KG - 1) / KG : 0;
    DigFrag<NP> f[3];
    auto fetch = [&](int st, DigFrag<NP>& to) {
        if (st < n_steps) {
            to.template load<0>(sa, sb);
            sa += a_adv;
            sb += b_adv;
        }
    };
    auto step = [&](int st, const DigFrag<NP>& cur, DigFrag<NP>& ahead) {
        if (st >= n_steps) return;
        fetch(st + 2, ahead);
        if (a_nar) {
#pragma unroll
            for (int i = 0; i < 4; ++i) row_nar |= pm_marker_bits((uint32_t)cur.a[NP - 1][i]);
        }
        if (b_nar) {
#pragma unroll
            for (int i = 0; i < 4; ++i) col_nar |= pm_marker_bits((uint32_t)cur.b[NP - 1][i]);
        }
        dig_mma<NP, 0, NP, 0, NP>(cur, acc);
    };
    fetch(0, f[0]);
    fetch(1, f[1]);
    for (int st = 0; st < n_steps; st += 3) {
        step(st, f[0], f[2]);
        step(st + 1, f[1], f[0]);
        step(st + 2, f[2], f[1]);
    }
    uint32_t* const rowv = lds + KG * L * 1024;  // [KG][32], then the columns'
    uint32_t* const colv = rowv + KG * 32;
    uint32_t* const vals = lds + kg * (L * 1024);
    row_nar = (row_nar | (uint32_t)__shfl_xor((int)row_nar, 32)) & 0x80808080u;
    col_nar = (col_nar | (uint32_t)__shfl_xor((int)col_nar, 32)) & 0x80808080u;
    if (lane < 32) {
        rowv[kg * 32 + lane] = row_nar;
        colv[kg * 32 + lane] = col_nar;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int lr = (r & 3) + 8 * (r >> 2) + 4 * (lane >> 5);
        uint32_t q[L];
        dig_combine<NP>(acc, r, q);
#pragma unroll
        for (int l = 0; l < L; ++l) vals[l * 1024 + lr * 32 + (lane & 31)] = q[l];
    }
    __syncthreads();
    const int col = t & 31, n = tn * 32 + col;
    if (n >= g.N) return;
    uint32_t cnar = 0;
#pragma unroll
    for (int k = 0; k < KG; ++k) cnar |= colv[k * 32 + col];
    auto value = [&](int lr, uint32_t (&q)[L]) {
#pragma unroll
        for (int l = 0; l < L; ++l) q[l] = lds[l * 1024 + (lr & 31) * 32 + col];
#pragma unroll
        for (int k = 1; k < KG; ++k) {
            uint32_t o[L];
#pragma unroll
            for (int l = 0; l < L; ++l) o[l] = lds[(k * L + l) * 1024 + (lr & 31) * 32 + col];
            quire_merge<L>(q, o);
        }
    };
    auto row_flag = [&](int lr) {
        uint32_t v = 0;
#pragma unroll
        for (int k = 0; k < KG; ++k) v |= rowv[k * 32 + (lr & 31)];
        return v;
    };
    const int rows = g.M - tm * 32 < 32 ? g.M - tm * 32 : 32;
    dig_round_column<L, 2 * KG>(g, at, tm * 32, n, t >> 5, rows, cnar, value, row_flag);
}

// Adds the slices of every output, adds the bias, rounds once.  One output per thread; the slices' limbs are read along
// the outputs.
template <int NP>
__device__ __forceinline__ void dig_merge(const DigGemmArgs& g) {
    constexpr int L = dig_limbs<NP>();
    const int64_t MN = (int64_t)g.M * g.N;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= MN) return;
    const int m = (int)(i / g.N), n = (int)(i - (int64_t)m * g.N);
    uint32_t q[L];
#pragma unroll
    for (int l = 0; l < L; ++l) q[l] = 0;
    uint32_t nar = 0;
    for (int z = 0; z < g.splits; ++z) {
        uint32_t o[L];
#pragma unroll
        for (int l = 0; l < L; ++l) o[l] = g.part[((int64_t)z * L + l) * MN + i];
        quire_merge<L>(q, o);
        nar |= g.rowflag[(int64_t)z * g.M + m] | g.colflag[(int64_t)z * g.N + n];
    }
    DigRound rd;
    rd.fin = g.fin;
    rd.fout = g.fout;
    rd.at = g.info->base[0] + g.info->base[1];
    const uint32_t bp = g.bias ? dig_load_pattern(g.bias, n, rd.fin.n) : 0u;
    dig_store_pattern(g.C, (int64_t)m * g.ldc + n, rd.fout.n, dig_round<L>(q, rd, nar != 0, g.bias != nullptr, bp));
}

// One launch for the slices of either plane count: NPA planes' in a, NPB planes' in b.
template <int NPA, int NPB>
__global__ __launch_bounds__(256) void dig_merge_kernel(DigGemmArgs a, DigGemmArgs b) {
    const int np = __builtin_amdgcn_readfirstlane(a.info->np);
    if (np == NPA && a.splits > 1) dig_merge<NPA>(a);
    if (NPB != NPA && np == NPB && b.splits > 1) dig_merge<NPB>(b);
}

// ---- host side ----

struct DigPlan {
    int RBA, RBB, KB;
    bool narrow;               // there is a kernel of NP1 planes in the call
    int splits, kb_per_split;  // of the kernel of NPS planes
    int wide_splits, wide_kb_per_split;  // of the one of NP2 planes behind a narrow one
    int kg;                    // groups of waves per workgroup in the kernel of NPS planes
    bool small;                // 32 x 32 tiles in the kernel of four planes
    size_t planes_bytes, ma_bytes, mb_bytes, stat_off, part_off, wide_part_off, total;
};

// posit(8,1): three planes (22 bits) hold what its Gaussian tensors use, and five sums leave room for a third wave per SIMD;
// below this size the second product kernel's launch costs more than that saves.
constexpr int64_t DIG_P8_1_NARROW = (int64_t)1 << 31;

// Most tiles of 64 x 64 for which the kernel of four planes takes 32 x 32 (us a call, posit(12,1), 64 -> 32): 8 tiles, K = 586 22.3 ->
// 17.2, 64 tiles, 512 21.2 -> 17.1, 96, 512 21.4 -> 19.5, 100, 640 23.2 -> 21.1; 144, 300 21.1 -> 21.9, 256, 1024 30.0 -> 34.8 (every
// operand is read twice as often).  Eight waves are slower than four from 65 tiles on (two workgroups on some compute units).
constexpr int DIG_SMALL_TILES = 112, DIG_SMALL_WAVES = 4;
// posit(8,1), whose reduction is never cut and whose older kernel leaves empty planes out: with more than one workgroup per compute
// unit only short reductions (us, 64 -> 32: 100 tiles, K = 512 18.7 -> 18.0, 1024 22.1 -> 23.6; 78, 640 20.3 -> 20.3, 8192 66 -> 94;
// 110, 448 18.6 -> 17.9, 768 20.5 -> 21.3; 112, 320 17.0 -> 16.8, 448 17.5 -> 18.2, 1024 22.0 -> 25.2; 250 workgroups, 8192 63.7 -> 61.0).
constexpr int DIG_SMALL_UNCUT_WGS = 256, DIG_SMALL_UNCUT_K = 320, DIG_SMALL_UNCUT_TILES = 110;
constexpr int64_t DIG_SMALL_UNCUT_TILES_K = 55000;

// The kernel that may always cut the reduction: that of four planes, or the only one.
template <class F>
constexpr int dig_nps() { return DigFormat<F>::NP1 == 4 ? 4 : DigFormat<F>::NP2; }

template <class F>
inline bool dig_small(int64_t M, int64_t N, int64_t K, int splits) {
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
    if (dig_nps<F>() != 4 || splits != 1) return false;
    if (F::N == 8 && !DigFormat<F>::BASE0)
        return ((M + 31) / 32) * ((N + 31) / 32) <= DIG_SMALL_UNCUT_WGS || (tiles <= DIG_SMALL_TILES && K <= DIG_SMALL_UNCUT_K) ||
               (tiles <= DIG_SMALL_UNCUT_TILES && tiles * K <= DIG_SMALL_UNCUT_TILES_K);
    return tiles <= DIG_SMALL_TILES;
}

// Room for 8 planes of both operands (posit(8,1): 4), the masks, 256 bytes for the decision, and what is not found inside
// on top: the scan's results take a slot that no kernel of posit(8,2) uses (posit(8,1): the rest of the 256 bytes), the partial sums of a cut reduction the slots
// that the narrow kernel leaves free if they fit there (posit(8,2): only then).  limit: bytes of workspace there may be.
template <class F>
inline DigPlan dig_plan(int64_t M, int64_t N, int64_t K, size_t limit = SIZE_MAX) {
    typedef DigFormat<F> D;
    constexpr int slots = F::N == 8 && !D::BASE0 ? D::NP2 : 8, NPS = dig_nps<F>();
    static_assert(sizeof(DigInfo) <= 32 && 32 + 2 * DIG_STAT_WGS8 * 2 <= 256, "decision and packed scan results");
    DigPlan p;
    const int64_t tm = (M + 63) / 64, tn = (N + 63) / 64, tiles = tm * tn;
    p.RBA = (int)tm * 2;
    p.RBB = (int)tn * 2;
    p.KB = (int)((K + 31) / 32);
    const size_t blocks = (size_t)p.KB * (p.RBA + p.RBB);
    p.planes_bytes = blocks * slots * 1024;
    p.ma_bytes = ((size_t)p.KB * p.RBA + 255) / 256 * 256;
    p.mb_bytes = ((size_t)p.KB * p.RBB + 255) / 256 * 256;
    p.total = p.planes_bytes + p.ma_bytes + p.mb_bytes + 256;
    p.stat_off = 0;
    if (dig_stat_packed<F>()) {
        p.stat_off = p.total - 256 + 32;
    } else if (F::N == 8) {
        p.stat_off = p.planes_bytes - DIG_STAT_BYTES;
    } else {
        p.stat_off = p.total;
        p.total += DIG_STAT_BYTES;
    }
    // Few tiles and a long reduction: slices, so that about 256 workgroups (one per compute unit) share it; each keeps at
    // least 16 k blocks, below which the merging launch costs more than it saves.
    const size_t rest = p.total;  // where partial sums go that find no room among the planes
    p.narrow = D::NP1 != 0 && (D::NP1 == 4 || M * N * K >= DIG_P8_1_NARROW);
    p.splits = 1;
    p.kb_per_split = p.KB;
    p.part_off = blocks * NPS * 1024;
    const size_t per = ((size_t)M * N * dig_limbs<NPS>() + M + N) * 4;
    int64_t s = 256 / tiles;
    if (s > p.KB / 16) s = p.KB / 16;
    if (s > 16) s = 16;
    if (F::N == 8 && s > (int64_t)((p.planes_bytes - p.part_off) / per)) s = (int64_t)((p.planes_bytes - p.part_off) / per);
    if (s > 1) {
        p.kb_per_split = (int)((p.KB + s - 1) / s);
        p.splits = (p.KB + p.kb_per_split - 1) / p.kb_per_split;
        if (p.splits * per > p.planes_bytes - p.part_off) {
            p.part_off = rest;
            p.total += p.splits * per;
        }
    }
    // The wide kernel takes four times as long per k block and two workgroups of half a tile fill a compute unit: slices of at least 8 k
    // blocks, where a merging launch is there anyway (all patterns of posit<16,1>, 96 x 97 x 4096: uncut 185 us, cut 39; 115 x 118 x 10332: 425 and 53).  posit(8,2)'s
    // fixed workspace has no room for them.
    p.wide_splits = 1;
    p.wide_kb_per_split = p.KB;
    p.wide_part_off = rest;
    if (D::NP1 == 4 && F::N != 8 && p.splits > 1) {
        int64_t w = 256 / tiles;
        if (w > p.KB / 8) w = p.KB / 8;
        if (w > 32) w = 32;
        const int kbps = (int)((p.KB + w - 1) / w), slices = (p.KB + kbps - 1) / kbps;
        const size_t total = rest + slices * (((size_t)M * N * dig_limbs<D::NP2>() + M + N) * 4);
        if (total <= limit) {
            p.wide_splits = slices;
            p.wide_kb_per_split = kbps;
            if (total > p.total) p.total = total;
        }
    }
    p.kg = NPS == 4 && tiles * p.splits <= 256 ? 2 : 1;
    p.small = dig_small<F>(M, N, K, p.splits);
    return p;
}

template <int NP, int KG>
inline hipError_t launch_dig_small(hipStream_t stream, DigGemmArgs g) {
    g.tiles_m = (g.M + 31) / 32;
    g.tiles_n = (g.N + 31) / 32;
    hipLaunchKernelGGL((dig_gemm_small_kernel<NP, KG>), dim3((unsigned)(g.tiles_m * g.tiles_n)), dim3(64 * KG), 0, stream, g);
    return hipGetLastError();
}

template <int NP, int KG, int S>
inline hipError_t launch_dig_product(hipStream_t stream, const DigGemmArgs& g, int splits) {
    hipLaunchKernelGGL((dig_gemm_kernel<NP, KG, S>), dim3((unsigned)(g.tiles_m * g.tiles_n), (unsigned)splits), dim3(256 * KG), 0, stream, g);
    return hipGetLastError();
}

// One group of waves per tile.  Four planes: dig_gemm_pair_kernel from the sizes on that fill the chip without cutting (us, dig_gemm_kernel and it: posit<16,1>
// 1500 x 700 x 2000 58.5 and 48.7, posit(8,2) 4096^3 508 and 478, (12,1) 3000 x 3000 x 300 68.7 and 62.1), but posit<16,1> beyond 2^35 multiply-adds, whose
// Gaussian operands reach the lowest plane in many pairs and few blocks (4096 x 4096 x 1024 200 and 195, 4096^3 652 and 680); three planes: dig_gemm_kernel
// (posit(8,1) 2500 x 1200 x 900 42.4 and 47.3).
template <int NP>
inline hipError_t launch_dig_whole(hipStream_t stream, DigGemmArgs g) {
    if constexpr (NP <= 4) {
        if (NP == 3 || (g.fin.n == 16 && (double)g.M * g.N * g.KB * 32 > (double)((int64_t)1 << 35))) return launch_dig_product<NP, 1, 4>(stream, g, g.splits);
    }
    if constexpr (NP >= 4) {
        g.tiles_n = (g.N + 31) / 32;
        const dim3 grid = dig_tile_grid((int64_t)g.tiles_m * g.tiles_n, g.splits);
        if (grid.z > 1) hipLaunchKernelGGL((dig_gemm_pair_kernel<NP, true>), grid, dim3(256), 0, stream, g);
        else hipLaunchKernelGGL((dig_gemm_pair_kernel<NP, false>), grid, dim3(256), 0, stream, g);
    }
    return hipGetLastError();
}

template <class F>
inline hipError_t launch_dig_gemm(hipStream_t stream, int transA, int transB, const void* A, int64_t lda, const void* B, int64_t ldb,
                                  const void* bias, void* C, int64_t ldc, int fout, int64_t M, int64_t N, int64_t K, void* workspace,
                                  size_t limit, const DigInfo** decision) {
    typedef DigFormat<F> D;
    constexpr int NPS = dig_nps<F>();
    const DigPlan p = dig_plan<F>(M, N, K, limit);
    uint8_t* base = (uint8_t*)workspace;
    uint8_t* ma = base + p.planes_bytes;
    uint8_t* mb = ma + p.ma_bytes;
    DigInfo* info = (DigInfo*)(mb + p.mb_bytes);
    void* stats = base + p.stat_off;
    *decision = info;
    const DigStatJob sa{A, transA ? K : M, transA ? M : K, lda, 0}, sb{B, transB ? N : K, transB ? K : N, ldb, 0};
    hipLaunchKernelGGL((dig_stat_kernel<F, dig_stat_packed<F>()>), dim3((unsigned)dig_stat_wgs<dig_stat_packed<F>()>(), 2), dim3(1024), 0, stream, sa, sb, stats);
    PNN_CHECK_LAUNCH();
    // op(A)[m,k] is A[m * lda + k] unless transA; op(B)[k,n] is B[k * ldb + n] unless transB
    const DigMatrixJob ja{A, transA ? (int64_t)1 : lda, transA ? lda : (int64_t)1, (int)M, (int)K, ma, p.RBA};
    const DigMatrixJob jb{B, transB ? ldb : (int64_t)1, transB ? (int64_t)1 : ldb, (int)N, (int)K, mb, p.RBB};
    const unsigned blocks0 = (unsigned)((p.RBA + 3) / 4) * (unsigned)p.KB, blocks1 = (unsigned)((p.RBB + 3) / 4) * (unsigned)p.KB;
    hipLaunchKernelGGL(dig_matrix_kernel<F>, dim3(blocks0 + blocks1), dim3(256), 0, stream, ja, jb, blocks0, stats, info, base, p.KB, p.narrow ? 1 : 0);
    PNN_CHECK_LAUNCH();
    DigGemmArgs g;
    g.planes = base; g.ma = ma; g.mb = mb; g.info = info;
    g.RBA = p.RBA; g.RBB = p.RBB; g.KB = p.KB;
    g.bias = bias; g.C = C; g.ldc = ldc;
    g.fin = fmt_of_code(code_of<F>()); g.fout = fmt_of_code(fout); g.M = (int)M; g.N = (int)N;
    g.tiles_m = p.RBA / 2;
    g.tiles_n = p.RBB / 2;
    auto slices = [&](int splits, int kb_per_split, size_t part_off, int limbs) {
        g.splits = splits;
        g.kb_per_split = kb_per_split;
        g.part = g.rowflag = g.colflag = nullptr;
        if (splits > 1) {
            g.part = (uint32_t*)(base + part_off);
            g.rowflag = g.part + (size_t)splits * limbs * M * N;
            g.colflag = g.rowflag + (size_t)splits * M;
        }
    };
    slices(p.splits, p.kb_per_split, p.part_off, dig_limbs<NPS>());
    hipError_t e;
    if constexpr (D::NP1 == 3) {
        if (p.narrow) {
            e = launch_dig_whole<D::NP1>(stream, g);
            if (e != hipSuccess) return e;
        }
    }
    if constexpr (NPS == 4) e = p.small ? launch_dig_small<4, DIG_SMALL_WAVES>(stream, g) : p.kg == 2 ? launch_dig_product<4, 2, 4>(stream, g, p.splits) : launch_dig_whole<4>(stream, g);
    else e = launch_dig_whole<NPS>(stream, g);
    if (e != hipSuccess) return e;
    const DigGemmArgs first = g;
    if constexpr (D::NP1 == 4) {
        slices(p.wide_splits, p.wide_kb_per_split, p.wide_part_off, dig_limbs<D::NP2>());
        e = launch_dig_whole<D::NP2>(stream, g);
        if (e != hipSuccess) return e;
    }
    if (p.splits > 1) {
        hipLaunchKernelGGL((dig_merge_kernel<NPS, D::NP2>), dim3((unsigned)((M * N + 255) / 256)), dim3(256), 0, stream, first, g);
        PNN_CHECK_LAUNCH();
    }
    return e;
}

}  // namespace pnn
