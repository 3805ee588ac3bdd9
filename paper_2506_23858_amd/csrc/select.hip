// vmoba_select: mean key blocks (Eq. 2), query x block similarities (Eq. 3), soft-max
// normalisation per query, head-global cumulative threshold (Eq. 4), TopkMask (Eq. 3) as a
// bit mask plus block-major and query-major sparse lists.
//
// The descending-sort-and-accumulate of Eq. 4 is done without sorting: P >= 0, so the order
// of its float bit patterns is the order of its values, and a three-level radix histogram
// (12 + 10 + 10 bits) with per-bin counts and per-bin sums locates the value theta at which
// the descending cumulative sum reaches tau * S.  Per-bin sums are kept as 64-bit integers
// (value * 2^fix_shift, truncated) so the result does not depend on the order of atomics.
#include "common.h"
#include "attn_common.h"

#include <algorithm>
#include <cmath>
#include <mutex>

namespace {

constexpr int HIST_BINS = 1024;
constexpr int QT = 64;          // queries per score tile
constexpr int SCAN_THREADS = 1024;
constexpr int SCAN_ITEMS = 16;

struct HeadState {              // one per (b, h), lives in the workspace
    unsigned long long need;    // fixed-point mass still missing inside the current bin range; after the last level: the position
                                // (row * blocks + block) of the last kept entry among those equal to theta, or TIE_RANKS
    unsigned long long cnt_above;  // pool entries strictly above the current bin range
    unsigned int prefix;        // float bits of theta found so far (high bits)
    unsigned int all;           // 1: threshold never reached -> keep every pair
    unsigned int n_tie;         // entries equal to theta (between the last two levels: candidates offered to the list)
    unsigned int take;          // how many of them belong to the top k (between the last two levels: 1 if a candidate was dropped)
};

// HeadState::need after the last level when the entries equal to theta have to be ranked row by row
constexpr unsigned long long TIE_RANKS = ~0ull;

struct SelectWs {               // workspace carve-up (device pointers)
    unsigned int* hist_cnt;         // [3][BH][1024]
    unsigned long long* hist_sum;   // [3][BH][1024]
    HeadState* state;               // [BH]
    int* ties;                      // [BH][S]   candidates of the last level, then (TIE_RANKS) per-row count of entries equal to theta
    int* tie_base;                  // [BH][S+1] exclusive scan of ties
    int* wtot;                      // [BH][n_waves]  pairs kept by each group of 64 queries, then its exclusive scan
    int* wcnt;                      // [BH][n_blocks][n_waves]
    int* row_tot;                   // [BH][n_blocks + 1]  totals of the rows of wcnt, then of wtot
    size_t zero_bytes;              // leading bytes (hist + state) cleared on every call
    float2* row_stat;   // [BH * S] {row maximum, row denominator} of the score soft-max (pool soft-max mode)
    float2* pool_stat;  // [BH] {pool maximum, 1 / pool denominator}
    size_t total;
};

SelectWs carve(void* base, int BH, int64_t S, int nb) {
    SelectWs w;
    char* p = (char*)base;
    size_t off = 0;
    w.hist_sum = (unsigned long long*)(p + off);  off += (size_t)3 * BH * HIST_BINS * 8;
    w.hist_cnt = (unsigned int*)(p + off);        off += (size_t)3 * BH * HIST_BINS * 4;
    w.state = (HeadState*)(p + off);              off += align_up((size_t)BH * sizeof(HeadState), 256);
    w.zero_bytes = off;
    w.ties = (int*)(p + off);                     off += align_up((size_t)BH * S * 4, 256);
    w.tie_base = (int*)(p + off);                 off += align_up((size_t)BH * (S + 1) * 4, 256);
    int64_t n_waves = ceil_div64(S, 64);
    w.wtot = (int*)(p + off);                     off += align_up((size_t)BH * n_waves * 4, 256);
    w.wcnt = (int*)(p + off);                     off += align_up((size_t)BH * nb * n_waves * 4, 256);
    w.row_tot = (int*)(p + off);                  off += align_up((size_t)BH * (nb + 1) * 4, 256);
    w.row_stat = (float2*)(p + off);              off += align_up((size_t)BH * S * 8, 256);
    w.pool_stat = (float2*)(p + off);             off += align_up((size_t)BH * 8, 256);
    w.total = off;
    return w;
}

// ---------------------------------------------------------------------------------------------
// Block means, Eq. 2.  One workgroup per (block, b*Hh + h).  Threads are laid out as
// (row group, 16-byte piece of a row); every thread sums its piece over the rows of its group,
// the groups are then added in a fixed order, so the result is reproducible.
// kv_rows: null when K is in block order, else the row of K that holds key position r (keys in place).
template <bool BF16, int D>
__global__ __launch_bounds__(256) void block_mean_kernel(TensorView K, const int* __restrict__ blk_off,
                                                         float* __restrict__ Bmean, int Hh, int nb,
                                                         const int* __restrict__ kv_rows,
                                                         unsigned int* __restrict__ zero_words, unsigned int n_zero) {
    constexpr int EPP = BF16 ? 8 : 4;          // elements per 16-byte piece
    constexpr int PIECES = D / EPP;            // pieces per row
    constexpr int GROUPS = 256 / PIECES;
    const int j = blockIdx.x, bh = blockIdx.y;
    const int b = bh / Hh, h = bh % Hh;
    {   // this workgroup's share of the words that must be zero when the next kernel of the call starts (histograms, state)
        const unsigned int n_wg = gridDim.x * gridDim.y, wg = bh * gridDim.x + j;
        const unsigned int per = (n_zero + n_wg - 1) / n_wg;
        const unsigned int z0 = min(n_zero, wg * per), z1 = min(n_zero, z0 + per);
        for (unsigned int i = z0 + threadIdx.x; i < z1; i += 256) zero_words[i] = 0u;
    }
    const int piece = threadIdx.x % PIECES, grp = threadIdx.x / PIECES;
    const int r0 = blk_off[j], r1 = blk_off[j + 1];
    float acc[EPP];
#pragma unroll
    for (int e = 0; e < EPP; ++e) acc[e] = 0.f;
    const char* base = K.ptr + ((long long)b * K.stride_b + (long long)h * K.stride_h) * (BF16 ? 2 : 4);
    for (int r = r0 + grp; r < r1; r += GROUPS) {
        const int row = kv_rows ? kv_rows[r] : r;
        const char* src = base + (long long)row * K.stride_s * (BF16 ? 2 : 4) + piece * 16;
        u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(src));
        if constexpr (BF16) {
            acc[0] += bf16lo_to_f32(v.x); acc[1] += bf16hi_to_f32(v.x);
            acc[2] += bf16lo_to_f32(v.y); acc[3] += bf16hi_to_f32(v.y);
            acc[4] += bf16lo_to_f32(v.z); acc[5] += bf16hi_to_f32(v.z);
            acc[6] += bf16lo_to_f32(v.w); acc[7] += bf16hi_to_f32(v.w);
        } else {
            acc[0] += __uint_as_float(v.x); acc[1] += __uint_as_float(v.y);
            acc[2] += __uint_as_float(v.z); acc[3] += __uint_as_float(v.w);
        }
    }
    __shared__ float red[GROUPS][D + 4];
#pragma unroll
    for (int e = 0; e < EPP; ++e) red[grp][piece * EPP + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < D) {
        float s = 0.f;
        for (int g = 0; g < GROUPS; ++g) s += red[g][threadIdx.x];
        Bmean[((long long)bh * nb + j) * D + threadIdx.x] = s / (float)(r1 - r0);
    }
}

// p * 2^fix_shift as an integer for a finite p >= 0 below 2^(63 - fix_shift), by a shift of the float's mantissa.
// Exact for every p whose last mantissa bit is worth at least 2^-fix_shift; smaller values (below 2^(-fix_shift + 23),
// at most 2^-14 of the pool's mass all together) count as 0.  Exactness is what lets a bin's sum be formed either value
// by value or as (count * leading bits + sum of trailing bits) << shift: both give the same integer.
__device__ __forceinline__ unsigned long long to_fixed(float p, int fix_shift) {
    const uint32_t b = __float_as_uint(p);
    const int e = (int)(b >> 23);
    const int sh = e - 150 + fix_shift;
    return (e && sh >= 0) ? ((unsigned long long)((b & 0x7fffffu) | 0x800000u) << sh) : 0ull;
}

// Level-0 histogram word in LDS: entries of one bin share sign, exponent and the three leading mantissa bits, so a bin
// needs only how many there are (bits 40..63) and the sum of their 20 trailing mantissa bits (bits 0..39): one 64-bit
// LDS atomic per entry.  Holds up to 2^20 entries per bin and workgroup.
constexpr unsigned long long PK_ONE = 1ull << 40;
// `copies` (a power of two) interleaved replicas of the 1024 words, word = bin * copies + (lane % copies): the entries of
// a row crowd into a few neighbouring bins, and lanes that hit the same word are served one after the other.
__device__ __forceinline__ void packed_hist_add(unsigned long long* sPk, int copy_shift, int copy, float p) {
    const unsigned int u = __float_as_uint(p);
    atomicAdd(&sPk[(min(u >> 20, (unsigned)(HIST_BINS - 1)) << copy_shift) + copy], PK_ONE | (unsigned long long)(u & 0xfffffu));
}
// A workgroup's packed words -> the head's level-0 histogram (count and fixed-point sum per bin).
__device__ __forceinline__ void packed_hist_flush(const unsigned long long* sPk, int copy_shift,
                                                  unsigned int* __restrict__ hist_cnt,
                                                  unsigned long long* __restrict__ hist_sum, long long bh, int fix_shift,
                                                  int tid, int n_threads) {
    for (int i = tid; i < HIST_BINS; i += n_threads) {
        unsigned long long cnt = 0, low = 0;
        for (int c = 0; c < (1 << copy_shift); ++c) {
            const unsigned long long w = sPk[(i << copy_shift) + c];
            cnt += w >> 40;
            low += w & (PK_ONE - 1);
        }
        if (cnt) {
            const int e = i >> 3, sh = e - 150 + fix_shift;
            const unsigned long long lead = 0x800000ull | ((unsigned long long)(i & 7) << 20);
            atomicAdd(&hist_cnt[bh * HIST_BINS + i], (unsigned int)cnt);
            if (e && sh >= 0) atomicAdd(&hist_sum[bh * HIST_BINS + i], (cnt * lead + low) << sh);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Scores (Eq. 3), row soft-max, P write-out and the first radix level, fused, for float32 queries
// (bfloat16 queries take score_mfma_kernel below).  A workgroup owns a tile of QT = 64 queries of
// one head.  The head's block means sit in LDS as float32; thread (q = tid % 64, g = tid / 64)
// keeps its query row in registers and computes the dot products with blocks g, g+4, g+8, ... and their exponentials; each of a row's four threads then
// adds all of them in the order of the blocks.  A tile of P is one flat run, written as such.
// Bound by its vector and LDS instructions.  2 heads x 512 tokens x 16 blocks 10.6 -> 7.7 us, selections of 12 x 14 040 x 36, 5 x 9360 x 180: 275 -> 261, 271 -> 257 us
// (before: every thread of a row computed all its exponentials, one wavefront wrote a row at a time, two LDS atomics per value).
template <int D>
__global__ __launch_bounds__(256) void score_kernel(TensorView Q, const float* __restrict__ Bmean,
                                                    float* __restrict__ P, unsigned int* __restrict__ hist_cnt,
                                                    unsigned long long* __restrict__ hist_sum,
                                                    int Hh, int S, int nb, float score_scale, int fix_shift,
                                                    float2* __restrict__ row_stat) {
    extern __shared__ __align__(16) unsigned char smem[];
    float* sB = reinterpret_cast<float*>(smem);                       // [nb][D]
    const int pstride = nb | 1;
    float* sP = sB + (size_t)nb * D;                                  // [QT][pstride]
    unsigned long long* sPk = reinterpret_cast<unsigned long long*>(sP + ((QT * pstride + 1) & ~1));   // [1024]
    float* sM = reinterpret_cast<float*>(sPk + HIST_BINS);            // [4][QT]

    const int bh = blockIdx.y;
    const int b = bh / Hh, h = bh % Hh;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;

    for (int i = tid; i < nb * D / 4; i += 256)
        reinterpret_cast<f32x4_t*>(sB)[i] = reinterpret_cast<const f32x4_t*>(Bmean + (long long)bh * nb * D)[i];
    for (int i = tid; i < HIST_BINS; i += 256) sPk[i] = 0ull;
    __syncthreads();

    const int n_tiles = (S + QT - 1) / QT;
    for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const int q0 = tile * QT;
        const int ql = lane;
        const int q = min(q0 + ql, S - 1);          // tail rows recompute the last query; never stored
        // query row -> registers
        float qr[D];
        {
            const char* src = Q.ptr + ((long long)b * Q.stride_b + (long long)q * Q.stride_s + (long long)h * Q.stride_h) * 4;
#pragma unroll
            for (int i = 0; i < D / 4; ++i) {
                f32x4_t v = reinterpret_cast<const f32x4_t*>(src)[i];
                qr[4 * i + 0] = v.x; qr[4 * i + 1] = v.y; qr[4 * i + 2] = v.z; qr[4 * i + 3] = v.w;
            }
        }
        float m = -INFINITY;
        for (int j = wave; j < nb; j += 4) {
            const f32x4_t* bj = reinterpret_cast<const f32x4_t*>(sB + (size_t)j * D);
            float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
            for (int i = 0; i < D / 4; ++i) {
                f32x4_t bv = bj[i];
                a0 = fmaf(qr[4 * i + 0], bv.x, a0);
                a1 = fmaf(qr[4 * i + 1], bv.y, a1);
                a2 = fmaf(qr[4 * i + 2], bv.z, a2);
                a3 = fmaf(qr[4 * i + 3], bv.w, a3);
            }
            const float x = ((a0 + a1) + (a2 + a3)) * score_scale;
            sP[ql * pstride + j] = x;
            m = fmaxf(m, x);
        }
        sM[wave * QT + ql] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) m = fmaxf(m, sM[w * QT + ql]);
        for (int j = wave; j < nb; j += 4) sP[ql * pstride + j] = expf(sP[ql * pstride + j] - m);
        __syncthreads();
        float den = 0.f;
        for (int j = 0; j < nb; ++j) den += sP[ql * pstride + j];
        if (row_stat && wave == 0 && q0 + ql < S) row_stat[(long long)bh * S + q0 + ql] = make_float2(m, den);
        __syncthreads();
        for (int j = wave; j < nb; j += 4) sP[ql * pstride + j] = sP[ql * pstride + j] / den;
        __syncthreads();
        // the [rows x nb] tile is a flat run of P; thread t writes its values t, t + 256, ... and enters them into the level-0 histogram
        const int rows = min(QT, S - q0);
        float* dst = P + ((long long)bh * S + q0) * nb;
        const int dr = 256 / nb, dj = 256 % nb;
        for (int e = tid, r = tid / nb, j = tid % nb; e < rows * nb; e += 256) {
            const float p = sP[r * pstride + j];
            dst[e] = p;
            if (hist_cnt) packed_hist_add(sPk, 0, 0, p);       // null: the caller takes the first radix level elsewhere (pool soft-max)
            r += dr;
            j += dj;
            if (j >= nb) { j -= nb; ++r; }
        }
        __syncthreads();
    }
    if (hist_cnt) packed_hist_flush(sPk, 0, hist_cnt, hist_sum, bh, fix_shift, tid, 256);
}

// ---------------------------------------------------------------------------------------------
// Scores on the matrix cores for bfloat16 queries (same results as score_kernel to float32
// rounding).  The float32 block means are split exactly into three bfloat16 terms,
// B = Bh + Bm + Bl (8 + 8 + 8 mantissa bits), so that every product with a bfloat16 query is exact
// in float32 and only the accumulation rounds -- a bfloat16 copy of the means alone would move P
// by ~4e-3.  S^T[block, q] = sum over the three terms of Bx[block, :] . Q[q, :], with the query on
// the MFMA column (= lane % 32), so the soft-max over blocks is a reduction over a lane's own
// registers plus one exchange with lane ^ 32.  SCORE_NW wavefronts x 32 queries per tile.
// With more than 189 blocks (192 at 64 channels) the three bfloat16 copies no longer fit the LDS; FLY keeps the means there as
// float32 (row stride D + 4) and splits every operand after its fetch: the same three terms from the same operations, so P is the
// same, at the price of vector work per matrix instruction.
// More than 256 blocks: score_long_kernel below.
// wavefronts per workgroup of the matrix-core score kernel (two per SIMD share one copy of the block means in LDS)
constexpr int SCORE_NW = 8, SCORE_NT = 64 * SCORE_NW, SCORE_QT = 32 * SCORE_NW;
// every value of a lane's rows (N_T tiles of 16) into the packed histogram
template <int N_T>
__device__ __forceinline__ void packed_hist_add_rows(unsigned long long* sPk, int copy_shift, int copy, const f32x16_t (&rows)[N_T], int n_mt) {
#pragma unroll
    for (int mt = 0; mt < N_T; ++mt) {
        if (mt < n_mt) {
#pragma unroll
            for (int v = 0; v < 16; ++v) packed_hist_add(sPk, copy_shift, copy, rows[mt][v]);
        }
    }
}
// Reduction over the 32 lanes of a wavefront half (lanes 0..31 and 32..63 separately): three steps inside rows of 16
// lanes by data-parallel primitives (quad swaps, half-row and row mirror), one across the half's two rows.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float half32_max(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    x = fmaxf(x, dpp_move<0xB1>(x));      // quad_perm [1, 0, 3, 2]
    x = fmaxf(x, dpp_move<0x4E>(x));      // quad_perm [2, 3, 0, 1]
    x = fmaxf(x, dpp_move<0x141>(x));     // row_half_mirror
    x = fmaxf(x, dpp_move<0x140>(x));     // row_mirror
    const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ float half32_sum(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    x += dpp_move<0xB1>(x);
    x += dpp_move<0x4E>(x);
    x += dpp_move<0x141>(x);
    x += dpp_move<0x140>(x);
    const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}
template <bool FIRST, class T>
__device__ __forceinline__ T& pick_ref(T& a, T& b) {
    if constexpr (FIRST) return a; else return b;
}
// NMT > 0: the number of 32-block tiles is that constant (a launch with terms picks the instantiation), so the
// loops over tiles carry no run-time tests and only the last tile knows padding blocks; NMT = 0 (FLY): read from nb.
// TR: the accumulators hold S^T (blocks down a lane's registers, the query on the lane: the soft-max of a row is in-lane,
// and a lane stores 16-byte runs of its row of P) -- for rows of P that start 16-byte aligned (N_b a multiple of 4), and FLY.
// !TR: they hold S (queries down the registers, the block on the lane): a store instruction then writes 128-byte runs of
// two rows with 4-byte pieces whatever N_b is, and the row maximum and sum take a reduction over 32 lanes.
template <int D, bool FLY, int NMT, bool TR>
__global__ __launch_bounds__(SCORE_NT) void score_mfma_kernel(TensorView Q, const float* __restrict__ Bmean,
                                                         float* __restrict__ P, unsigned int* __restrict__ hist_cnt,
                                                         unsigned long long* __restrict__ hist_sum,
                                                         int BH, int Hh, int S, int nb, float score_scale,
                                                         int fix_shift, int copy_shift, float2* __restrict__ row_stat) {
    // LDS rows of the bf16 terms are padded by 16 bytes.  Beyond 128 blocks (NMT > 4) only the nb real rows and one row of
    // zeros are kept -- the lanes of the last tile that stand for padding blocks read the zero row -- which is what lets
    // three terms of up to 189 blocks fit beside the histogram words.
    constexpr bool CLAMP = NMT > 4;
    constexpr int STR = D + 8;                 // LDS row stride in bf16 elements
    constexpr int FSTR = D + 4;                // LDS row stride in float elements (FLY)
    constexpr int KSTEPS = D / 16;
    static_assert(FLY == (NMT == 0) && !(FLY && !TR), "one launch with float32 means, or terms of a known number of tiles");
    constexpr int MAX_MT = FLY ? 8 : NMT;                        // FLY: up to 256 blocks
    extern __shared__ __align__(16) unsigned char smem[];
    const int nb_pad = NMT > 0 ? NMT * 32 : ((nb + 31) & ~31);
    const int n_mt = NMT > 0 ? NMT : nb_pad / 32;
    const int n_rows = CLAMP ? nb + 1 : nb_pad;                   // rows of a term in LDS
    auto term_at = [&](int x, int row, int el) { return ((size_t)x * n_rows + row) * STR + el; };
    __bf16* sB = reinterpret_cast<__bf16*>(smem);                                  // [3][n_rows][STR]
    float* sBf = reinterpret_cast<float*>(smem);                                   // FLY: [nb_pad][FSTR]
    unsigned long long* sPk = FLY ? reinterpret_cast<unsigned long long*>(sBf + (size_t)nb_pad * FSTR)
                                  : reinterpret_cast<unsigned long long*>(sB + (size_t)3 * n_rows * STR);   // [1024 << copy_shift]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hf = lane >> 5;
    const int hist_copy = lane & ((1 << copy_shift) - 1);

    // block means of head bh -> LDS, 16 bytes per lane and four loads in flight per lane (the head's means are one
    // contiguous array); clears the histogram words
    auto load_means = [&](int bh) {
        const f32x4_t* src4 = reinterpret_cast<const f32x4_t*>(Bmean + (long long)bh * nb * D);
        const int n4 = nb * D / 4, n4_pad = (FLY ? nb_pad : n_rows) * D / 4;      // rows past nb are zeros
        for (int i0 = tid; i0 < n4_pad; i0 += 4 * SCORE_NT) {
            f32x4_t x4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * SCORE_NT;
                const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
                x4[u] = i < n4 ? src4[i] : z;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * SCORE_NT;
                if (i >= n4_pad) continue;
                const int j = (i * 4) / D, d = (i * 4) % D;
                if constexpr (FLY) {
                    *reinterpret_cast<f32x4_t*>(&sBf[j * FSTR + d]) = x4[u];
                } else {
                    bf16x4_t h4, m4, l4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = x4[u][e];
                        const __bf16 xh = (__bf16)x;
                        const float r1 = x - (float)xh;
                        const __bf16 xm = (__bf16)r1;
                        const float r2 = r1 - (float)xm;
                        h4[e] = xh;
                        m4[e] = xm;
                        l4[e] = (__bf16)r2;
                    }
                    *reinterpret_cast<bf16x4_t*>(&sB[term_at(0, j, d)]) = h4;
                    *reinterpret_cast<bf16x4_t*>(&sB[term_at(1, j, d)]) = m4;
                    *reinterpret_cast<bf16x4_t*>(&sB[term_at(2, j, d)]) = l4;
                }
            }
        }
        for (int i = tid; i < (HIST_BINS << copy_shift); i += SCORE_NT) sPk[i] = 0ull;
    };

    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int n_tiles = (S + SCORE_QT - 1) / SCORE_QT;
    const bool vec_ok = (nb & 3) == 0;                       // a row of P starts 16-byte aligned
    // The launch's work is the flat list of (head, query tile) pairs; a workgroup takes one contiguous share of it, so
    // all shares are equal to within one tile whatever the number of heads, and reloads the means when its share
    // crosses into the next head.
    const int n_flat = BH * n_tiles;
    const int t0 = (int)((long long)blockIdx.x * n_flat / gridDim.x), t1 = (int)((long long)(blockIdx.x + 1) * n_flat / gridDim.x);
    auto load_q = [&](int flat, bf16x8_t(&dst)[KSTEPS]) {
        const int bh = flat / n_tiles, tile = flat - bh * n_tiles, b = bh / Hh, h = bh - b * Hh;
        const int qc = min(tile * SCORE_QT + wave * 32 + l32, S - 1);     // rows past the end recompute the last query; never stored
        const char* src = Q.ptr + ((long long)b * Q.stride_b + (long long)qc * Q.stride_s + (long long)h * Q.stride_h) * 2;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) dst[ks] = *reinterpret_cast<const bf16x8_t*>(src + (ks * 16 + hf * 8) * 2);
    };
    // Order inside a tile: request the next tile's query rows, matrix phase, soft-max arithmetic, then -- only then --
    // wait for the rows requested a whole tile ago, take them over and store this tile's P.  The stores then drain during
    // the next tile's arithmetic.  The take-over is written as opaque register moves: as a plain assignment the compiler
    // turns it into the loop-carried copy at the bottom of the loop, behind the stores, and its wait for the rows there
    // becomes a wait for every store just issued.
    bf16x8_t qf[KSTEPS], qn[KSTEPS];
    constexpr bool EARLY_ROWS = NMT > 0 && NMT <= 4;                  // see the tile loop
    auto take_next_rows = [&]() {
        if constexpr (!EARLY_ROWS) return;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const u32x4_t src = __builtin_bit_cast(u32x4_t, qn[ks]);
            unsigned int d0, d1, d2, d3;
            asm volatile("v_mov_b32 %0, %4\n\tv_mov_b32 %1, %5\n\tv_mov_b32 %2, %6\n\tv_mov_b32 %3, %7"
                         : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3)
                         : "v"(src.x), "v"(src.y), "v"(src.z), "v"(src.w));
            const u32x4_t dst = {d0, d1, d2, d3};
            qf[ks] = __builtin_bit_cast(bf16x8_t, dst);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if (t0 < t1) {                                       // the first tile's rows come the same way (the matrix phase then
        if constexpr (EARLY_ROWS) {                      // never reads a register that a load is still to fill)
            load_q(t0, qn);
            take_next_rows();
        } else {
            load_q(t0, qf);
        }
    }
    int cur_bh = -1, since_flush = 0;
    const int flush_every = max(1, (1 << 20) / (SCORE_QT * nb_pad));   // tiles until a packed histogram word could overflow
    // A tile's P values stay in `outp` until the NEXT tile's matrix phase is over and are entered into the histogram only
    // then.  That keeps them in registers of their own: the matrix phase then writes accumulators that no store still
    // in flight reads (the compiler makes a wavefront wait for such stores before it overwrites their data).
    // (With more than 3 tiles of accumulators there are no registers for a second set: the values stay in the
    // accumulators and are counted right after their stores.)
    constexpr bool DEFER = NMT > 0 && NMT <= 3;
    f32x16_t outp_own[MAX_MT] = {};                                  // never touched unless DEFER
    bool pending = false;                                             // this lane's outp holds a query's row not yet counted
    const bool count = hist_cnt != nullptr;
    for (int flat = t0; flat < t1; ++flat) {
        const int bh = flat / n_tiles, tile = flat - bh * n_tiles;
        if (bh != cur_bh || since_flush >= flush_every) {              // same decision in every wavefront
            since_flush = 0;
            if (cur_bh >= 0) {
                if (DEFER && count && pending) packed_hist_add_rows<MAX_MT>(sPk, copy_shift, hist_copy, outp_own, n_mt);
                pending = false;
                __syncthreads();
                if (hist_cnt) packed_hist_flush(sPk, copy_shift, hist_cnt, hist_sum, cur_bh, fix_shift, tid, SCORE_NT);
                __syncthreads();
            }
            load_means(bh);
            __syncthreads();
            cur_bh = bh;
        }
        ++since_flush;
        const int q = tile * SCORE_QT + wave * 32 + l32;
        // the next tile's rows: requested here, a whole tile before their use, where the registers allow (up to four
        // 32-block tiles); else after the matrix phase, which leaves the soft-max arithmetic for them to arrive
        if constexpr (EARLY_ROWS) {
            load_q(min(flat + 1, t1 - 1), qn);
            __builtin_amdgcn_sched_barrier(0);                        // requested here, not after the matrix phase
        }
        f32x16_t acc[MAX_MT];
#pragma unroll
        for (int mt = 0; mt < MAX_MT; ++mt) acc[mt] = zero16;
        // k-step outermost: consecutive matrix instructions go to different accumulators (each accumulator still sums
        // its terms in the order k-step, then high / middle / low part)
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
#pragma unroll
            for (int mt = 0; mt < MAX_MT; ++mt) {
                if (mt < n_mt) {
                    if constexpr (FLY) {
                        const float* src = &sBf[(mt * 32 + l32) * FSTR + ks * 16 + hf * 8];
                        const f32x4_t x0 = *reinterpret_cast<const f32x4_t*>(src), x1 = *reinterpret_cast<const f32x4_t*>(src + 4);
                        bf16x8_t bh8, bm8, bl8;
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const float x = i < 4 ? x0[i] : x1[i - 4];
                            const __bf16 xh = (__bf16)x;
                            const float r1 = x - (float)xh;
                            const __bf16 xm = (__bf16)r1;
                            const float r2 = r1 - (float)xm;
                            bh8[i] = xh;
                            bm8[i] = xm;
                            bl8[i] = (__bf16)r2;
                        }
                        acc[mt] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bh8, qf[ks], acc[mt], 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], bh8, acc[mt], 0, 0, 0);
                        acc[mt] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bm8, qf[ks], acc[mt], 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], bm8, acc[mt], 0, 0, 0);
                        acc[mt] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bl8, qf[ks], acc[mt], 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], bl8, acc[mt], 0, 0, 0);
                    }
                }
            }
            if constexpr (!FLY) {
                // a batch of fragments is requested before its first matrix instruction, so one LDS latency is paid per
                // batch, not per instruction; the whole k-step is one batch where the registers allow it
                constexpr int XB = (NMT > 0 && NMT <= 3) ? 3 : 1;
#pragma unroll
                for (int x0 = 0; x0 < 3; x0 += XB) {
                    bf16x8_t bf[XB][MAX_MT];
#pragma unroll
                    for (int x = 0; x < XB; ++x)
#pragma unroll
                        for (int mt = 0; mt < MAX_MT; ++mt)
                            if (mt < n_mt)
                                bf[x][mt] = *reinterpret_cast<const bf16x8_t*>(
                                    &sB[term_at(x0 + x, (CLAMP && mt == NMT - 1) ? min(mt * 32 + l32, nb) : mt * 32 + l32, ks * 16 + hf * 8)]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int x = 0; x < XB; ++x)
#pragma unroll
                        for (int mt = 0; mt < MAX_MT; ++mt)
                            if (mt < n_mt) acc[mt] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[x][mt], qf[ks], acc[mt], 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], bf[x][mt], acc[mt], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!EARLY_ROWS) {                                  // straight into the registers the matrix phase has just freed
            load_q(min(flat + 1, t1 - 1), qf);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (DEFER && count && pending) packed_hist_add_rows<MAX_MT>(sPk, copy_shift, hist_copy, outp_own, n_mt);   // the previous tile's row
        pending = false;
        // accumulator value v of tile mt <-> block 32*mt + 8*(v>>2) + 4*hf + (v&3) = 32*mt + 4*hf + c(v).  A value is a
        // real block (not padding up to the tile) when c(v) < lim, lim = nb - 32*mt - 4*hf; a whole group of four
        // consecutive blocks when c(v) + 3 < lim.  With NMT fixed, every tile but the last is all real blocks.
        auto tile_full = [&](int mt) { return NMT > 0 && mt < NMT - 1; };
        if constexpr (!TR) {
            // accumulator value v of tile mt <-> query row 8*(v>>2) + 4*hf + (v&3) of the wavefront's 32, block 32*mt + l32
            const int q_w = tile * SCORE_QT + wave * 32 + 4 * hf;         // + 8*(v>>2) + (v&3)
            float* prow = P + ((long long)bh * S + q_w) * nb + l32;
            auto col_ok = [&](int mt) { return tile_full(mt) || mt * 32 + l32 < nb; };
            float mrow[16], den[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float t = -INFINITY;
#pragma unroll
                for (int mt = 0; mt < MAX_MT; ++mt) {
                    if (mt < n_mt) {
                        float sv = acc[mt][v] * score_scale;
                        if (!tile_full(mt)) sv = col_ok(mt) ? sv : -INFINITY;
                        acc[mt][v] = sv;
                        t = fmaxf(t, sv);
                    }
                }
                mrow[v] = half32_max(t);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float d = 0.f;
#pragma unroll
                for (int mt = 0; mt < MAX_MT; ++mt) {
                    if (mt < n_mt) {
                        const float e = __builtin_amdgcn_exp2f((acc[mt][v] - mrow[v]) * 1.44269504088896340736f);
                        acc[mt][v] = e;
                        d += e;
                    }
                }
                den[v] = half32_sum(d);
            }
            take_next_rows();
            auto& outp = pick_ref<DEFER>(outp_own, acc);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int dq = 8 * (v >> 2) + (v & 3);
                const bool live = q_w + dq < S;                   // a row past the end repeats the last query: counted as zeros
                const float inv_den = 1.f / den[v];
                if (row_stat && live && l32 == 0) row_stat[(long long)bh * S + q_w + dq] = make_float2(mrow[v], den[v]);
#pragma unroll
                for (int mt = 0; mt < MAX_MT; ++mt)
                    if (mt < n_mt) outp[mt][v] = live ? acc[mt][v] * inv_den : 0.f;
            }
#pragma unroll
            for (int mt = 0; mt < MAX_MT; ++mt) {
                if (mt < n_mt && col_ok(mt)) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int dq = 8 * (v >> 2) + (v & 3);
                        if (q_w + dq < S) prow[(long long)dq * nb + mt * 32] = outp[mt][v];
                    }
                }
            }
            // padding blocks and rows past the end hold P = 0 and land in bin 0 (see below)
            if constexpr (DEFER) pending = true;
            else if (count) packed_hist_add_rows<MAX_MT>(sPk, copy_shift, hist_copy, acc, n_mt);
            continue;
        }
        float m = -INFINITY;
#pragma unroll
        for (int mt = 0; mt < MAX_MT; ++mt) {
            if (mt < n_mt) {
                const int lim = nb - 32 * mt - 4 * hf;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float sv = acc[mt][v] * score_scale;
                    if (!tile_full(mt)) sv = (8 * (v >> 2) + (v & 3) < lim) ? sv : -INFINITY;
                    acc[mt][v] = sv;
                    m = fmaxf(m, sv);
                }
            }
        }
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        // exp(x) for x <= 0 as 2^(x * log2 e): one rounding in the product (relative error of the result below
        // 1e-7 * |x|, i.e. an absolute error below 1e-7 on every P that is not itself negligible) and the hardware's
        // 2^x (1 ulp); exp(-inf) = 0 on padding blocks
        float den = 0.f;
#pragma unroll
        for (int mt = 0; mt < MAX_MT; ++mt) {
            if (mt < n_mt) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float e = __builtin_amdgcn_exp2f((acc[mt][v] - m) * 1.44269504088896340736f);
                    acc[mt][v] = e;
                    den += e;
                }
            }
        }
        den += __shfl_xor(den, 32, 64);
        take_next_rows();
        auto& outp = pick_ref<DEFER>(outp_own, acc);
        {
            const float inv_den = 1.f / den;
#pragma unroll
            for (int mt = 0; mt < MAX_MT; ++mt)
                if (mt < n_mt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) outp[mt][v] = acc[mt][v] * inv_den;
        }
        if (row_stat && q < S && hf == 0) row_stat[(long long)bh * S + q] = make_float2(m, den);
        if (q < S) {
            float* dst = P + ((long long)bh * S + q) * nb;
#pragma unroll
            for (int mt = 0; mt < MAX_MT; ++mt) {
                if (mt < n_mt) {
                    const int lim = nb - 32 * mt - 4 * hf;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int j0 = mt * 32 + 8 * g + 4 * hf;
                        if (vec_ok && (tile_full(mt) || 8 * g + 3 < lim)) {
                            const f32x4_t o = {outp[mt][4 * g], outp[mt][4 * g + 1], outp[mt][4 * g + 2], outp[mt][4 * g + 3]};
                            *reinterpret_cast<f32x4_t*>(dst + j0) = o;
                        } else {
#pragma unroll
                            for (int r = 0; r < 4; ++r) if (8 * g + r < lim) dst[j0 + r] = outp[mt][4 * g + r];
                        }
                    }
                }
            }
        }
        // first radix level, deferred: padding blocks hold P = 0 and land in bin 0 with the true zeros; that bin has no mass
        // and is the last of the descending scan, so neither a cut by mass nor one by count ever looks at its count.
        if constexpr (DEFER) pending = q < S;
        else if (count && q < S) packed_hist_add_rows<MAX_MT>(sPk, copy_shift, hist_copy, acc, n_mt);
    }
    if (DEFER && count && pending) packed_hist_add_rows<MAX_MT>(sPk, copy_shift, hist_copy, outp_own, n_mt);
    __syncthreads();
    if (hist_cnt && cur_bh >= 0) packed_hist_flush(sPk, copy_shift, hist_cnt, hist_sum, cur_bh, fix_shift, tid, SCORE_NT);
}

// ---------------------------------------------------------------------------------------------
// More than 256 blocks.  A query's scores stay in the registers, NMT tiles of 32 blocks; what does not fit is the block means in LDS, so
// they pass through it, 64 blocks at a time in two buffers (split into the same three terms by the threads that bring them: 147 KB per
// 128 channels, 288 blocks and tile, from the L2).  Accumulators as in score_mfma_kernel without TR: the block on the lane, 16 rows down the registers.
// The soft-max has the operations, and the sums the order, of one wavefront per row whose lane owns columns lane, lane + 64, ...:
// den = the two halves' sums over the even and the odd tiles, then lanes 16, 8, 4, 2, 1 apart.
// NW wavefronts of 32 queries each: 8 while NMT tiles leave two wavefronts per SIMD enough registers (NMT = 9), else 4.
// Bound by its vector instructions, 49 per value: a quarter expf, then the histogram's word, the quotient, the reductions.  12 heads x 112 320 tokens x 288 blocks
// (selection 2.87 -> 2.2 ms): 0.70 ms; before, launches for 144 blocks each wrote the scores (0.67) and another normalised them in place (0.68), 4.6 GB instead of
// 1.55.  Selections of 128 channels, 8 heads x 33 K tokens x 264 blocks, 8 x 106 K x 300 and 330, 12 x 115 K x 400, 12 x 98 K x 512: 0.49 / 1.99 / 2.34 / 4.24 / 4.43 -> 0.38 / 1.59 / 1.92 /
// 3.81 / 4.07 ms; of 64, 12 heads x 115 K tokens x 384 and 448 blocks, 98 K x 512: 3.79 / 4.45 / 4.32 -> 3.07 / 3.53 / 3.60.  Same bits.  The gain is smallest where registers do not suffice:
// 14 tiles of 128 channels and 16 of either spill 23 to 69, beside a wavefront's copies to and from accumulator registers.
// Values below any possible theta left out of the histogram: no gain; expf without its test for an overflow: none.
constexpr int LONG_KB = 64;                             // blocks per LDS buffer
constexpr int LONG_COPIES = 2;                          // log2 of the histogram's replicas
template <int CTRL>
__device__ __forceinline__ float dpp_ror(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true)); }
template <int D, int NMT, int NW>
__global__ __launch_bounds__(64 * NW, NW / 4) void score_long_kernel(TensorView Q, const float* __restrict__ Bmean, float* __restrict__ P,
                                                                     unsigned int* __restrict__ hist_cnt, unsigned long long* __restrict__ hist_sum, int BH, int Hh,
                                                                     int S, int nb, float score_scale, int fix_shift, float2* __restrict__ row_stat) {
    constexpr int STR = D + 8, KSTEPS = D / 16, NT = 64 * NW, TQ = 32 * NW, COPIES = LONG_COPIES;
    constexpr int NCH = (NMT + 1) / 2, TERM = LONG_KB * STR, BUF = 3 * TERM;         // chunks; elements of a term and of a buffer
    constexpr int NLD = LONG_KB * D / 4 / NT;                                         // 16-byte pieces of means per thread and chunk
    static_assert(NLD * NT * 4 == LONG_KB * D, "equal shares");
    extern __shared__ __align__(16) unsigned char smem[];
    __bf16* sB = reinterpret_cast<__bf16*>(smem);                                     // [2][3][LONG_KB][STR]
    unsigned long long* sPk = reinterpret_cast<unsigned long long*>(sB + 2 * BUF);    // [HIST_BINS << COPIES]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hf = lane >> 5, copy = lane & ((1 << COPIES) - 1);
    const int n_tiles = (S + TQ - 1) / TQ, n_flat = BH * n_tiles;
    const int t0 = (int)((long long)blockIdx.x * n_flat / gridDim.x), t1 = (int)((long long)(blockIdx.x + 1) * n_flat / gridDim.x);
    if (t0 >= t1) return;
    bf16x8_t qf[KSTEPS];
    auto load_q = [&](int flat) {
        const int bh = flat / n_tiles, tile = flat - bh * n_tiles, b = bh / Hh, h = bh - b * Hh;
        const int qc = min(tile * TQ + wave * 32 + l32, S - 1);           // rows past the end recompute the last query; never stored
        const char* src = Q.ptr + ((long long)b * Q.stride_b + (long long)qc * Q.stride_s + (long long)h * Q.stride_h) * 2;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8_t*>(src + (ks * 16 + hf * 8) * 2);
    };
    f32x4_t mean[NLD];
    auto load_means = [&](int bh, int c) {                                // blocks past the last are zeros
        const f32x4_t* src = reinterpret_cast<const f32x4_t*>(Bmean + ((long long)bh * nb + c * LONG_KB) * D);
        const int n4 = (nb - c * LONG_KB) * (D / 4);
        const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < NLD; ++u) mean[u] = tid + u * NT < n4 ? src[tid + u * NT] : z;
    };
    auto store_means = [&](int buf) {
#pragma unroll
        for (int u = 0; u < NLD; ++u) {
            const int i = (tid + u * NT) * 4;
            __bf16* dst = sB + buf * BUF + i / D * STR + i % D;
            u32x2_t t[3];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float x0 = mean[u][2 * e], x1 = mean[u][2 * e + 1];
                t[0][e] = pack_bf16x2(x0, x1);
                const float r0 = x0 - bf16lo_to_f32(t[0][e]), r1 = x1 - bf16hi_to_f32(t[0][e]);
                t[1][e] = pack_bf16x2(r0, r1);
                t[2][e] = pack_bf16x2(r0 - bf16lo_to_f32(t[1][e]), r1 - bf16hi_to_f32(t[1][e]));
            }
#pragma unroll
            for (int x = 0; x < 3; ++x) *reinterpret_cast<u32x2_t*>(dst + x * TERM) = t[x];
        }
    };
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int flush_every = max(1, (1 << 20) / (TQ * NMT * 32));          // tiles until a packed histogram word could overflow
    int cur_bh = t0 / n_tiles, since_flush = 0, buf = 0;
    for (int i = tid; i < (HIST_BINS << COPIES); i += NT) sPk[i] = 0ull;
    load_q(t0);
    load_means(cur_bh, 0);
    store_means(0);
    for (int flat = t0; flat < t1; ++flat) {
        const int bh = flat / n_tiles, tile = flat - bh * n_tiles;
        if (hist_cnt && (bh != cur_bh || since_flush >= flush_every)) {   // same decision in every wavefront
            __syncthreads();
            packed_hist_flush(sPk, COPIES, hist_cnt, hist_sum, cur_bh, fix_shift, tid, NT);
            __syncthreads();
            for (int i = tid; i < (HIST_BINS << COPIES); i += NT) sPk[i] = 0ull;
            since_flush = 0;
        }
        cur_bh = bh;
        ++since_flush;
        f32x16_t acc[NMT];
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt) acc[mt] = zero16;
        const int next = min(flat + 1, t1 - 1);
        static_for<NCH>([&](auto cc) __attribute__((always_inline)) {
            constexpr int c = cc, N = c * 2 + 1 < NMT ? 2 : 1;            // tiles of the chunk
            __syncthreads();                                              // chunk c is in the LDS; everybody is done with the one before
            load_means(c + 1 < NCH ? bh : next / n_tiles, c + 1 < NCH ? c + 1 : 0);
            const __bf16* src = sB + buf * BUF + l32 * STR + hf * 8;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                bf16x8_t b[3][N];
#pragma unroll
                for (int x = 0; x < 3; ++x)
#pragma unroll
                    for (int t = 0; t < N; ++t) b[x][t] = *reinterpret_cast<const bf16x8_t*>(src + x * TERM + t * 32 * STR + ks * 16);
#pragma unroll
                for (int x = 0; x < 3; ++x)
#pragma unroll
                    for (int t = 0; t < N; ++t) acc[c * 2 + t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], b[x][t], acc[c * 2 + t], 0, 0, 0);
            }
            store_means(buf ^ 1);
            buf ^= 1;
        });
        load_q(next);
        __builtin_amdgcn_sched_barrier(0);
        // accumulator value v of tile mt <-> query row 8*(v>>2) + 4*hf + (v&3) of the wavefront's 32, block 32*mt + l32
        const int q_w = tile * TQ + wave * 32 + 4 * hf;
        float* prow = P + ((long long)bh * S + q_w) * nb + l32;
        const bool whole = tile * TQ + wave * 32 + 32 <= S;
        auto col_ok = [&](int mt) { return mt < 8 || mt * 32 + l32 < nb; };           // (more than 256 blocks)
        auto batch = [&](int v0) __attribute__((always_inline)) {                     // rows of four accumulator values
            float m[4], den[4], rcp[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float t = -INFINITY;
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    float sv = acc[mt][v0 + i] * score_scale;
                    asm("" : "+v"(sv));                                  // rounded here: not to become a part of sv - m
                    if (mt >= 8) sv = col_ok(mt) ? sv : -INFINITY;
                    acc[mt][v0 + i] = sv;
                    t = fmaxf(t, sv);
                }
                m[i] = half32_max(t);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float d[2] = {0.f, 0.f};
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    const float e = expf(acc[mt][v0 + i] - m[i]);         // exp(-inf) = 0 past the row's end
                    acc[mt][v0 + i] = e;
                    d[mt & 1] += e;
                }
                float x = d[0] + d[1];
                typedef unsigned u2 __attribute__((ext_vector_type(2)));
                const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                x = __uint_as_float(r.x) + __uint_as_float(r.y);
                x += dpp_ror<0x128>(x);
                x += dpp_ror<0x124>(x);
                x += dpp_ror<0x122>(x);
                x += dpp_ror<0x121>(x);
                den[i] = x * 0x1p64f;
                rcp[i] = 1.f / x * 0x1p-64f;
                if constexpr (NMT == 16) __builtin_amdgcn_sched_barrier(0);      // (rows overlapped: five times the scratch accesses at 64 channels)
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int dq = 2 * v0 + i;                                // = 8 * (v >> 2) + (v & 3)
                const bool live = whole || q_w + dq < S;
                if (row_stat && live && l32 == 0) row_stat[(long long)bh * S + q_w + dq] = make_float2(m[i], den[i] * 0x1p-64f);
#pragma unroll
                for (int mt = 0; mt < NMT; ++mt) {
                    // the quotient, correctly rounded: from a correctly rounded reciprocal one correction step is enough (P. Markstein, IBM J. Res. Dev. 34, 1990)
                    // if the remainder is exact, hence the 2^64: without it, it is not for exponentials below 2^-102
                    const float e = acc[mt][v0 + i] * 0x1p64f, q0 = e * rcp[i], p = fmaf(fmaf(-q0, den[i], e), rcp[i], q0);
                    if (live && (mt < 8 || col_ok(mt))) {
                        prow[(long long)dq * nb + mt * 32] = p;
                        if (hist_cnt) packed_hist_add(sPk, COPIES, copy, p);
                    }
                }
            }
        };
#pragma unroll
        for (int v0 = 0; v0 < 16; v0 += 4) {
            batch(v0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();
    if (hist_cnt) packed_hist_flush(sPk, COPIES, hist_cnt, hist_sum, cur_bh, fix_shift, tid, NT);
}

// ---------------------------------------------------------------------------------------------
// Descending scan of one radix level.  One workgroup of 1024 threads per head; thread t owns
// bin 1023 - t, so an inclusive prefix sum over t is the descending cumulative sum.
// BYCOUNT = false: the cut is where the descending cumulative SUM reaches `target` (threshold selection,
// Eq. 4); BYCOUNT = true: where the descending cumulative COUNT reaches it (a fixed global k).
// The cut inside one level's bins, by 1024 threads: my_s / my_c = mass and count of bin 1023 - t.  Returns true in the one thread whose
// bin holds the cut (level 0: or in the last thread when the pool does not reach the target), with the new state in *st.
struct ScanLds { unsigned long long s[HIST_BINS / 64]; unsigned int c[HIST_BINS / 64]; };
static_assert(HIST_BINS / 64 == 16, "scan_level sums over wavefronts in a row of 16 lanes");
// Inclusive prefix sums over the 64 lanes, or over each row of 16, by data-parallel-primitive moves: a shuffle is a trip through the LDS,
// two for 64 bits.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned int moved32(unsigned int x) { return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false); }
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long moved64(unsigned long long x) {
    return (unsigned long long)moved32<CTRL, ROWS>((unsigned int)(x >> 32)) << 32 | moved32<CTRL, ROWS>((unsigned int)x);
}
constexpr int ROW_SHR = 0x110, ROW_BCAST15 = 0x142, ROW_BCAST31 = 0x143;
__device__ __forceinline__ unsigned int row_scan32(unsigned int x) {
    x += moved32<ROW_SHR + 1, 0xf>(x);
    x += moved32<ROW_SHR + 2, 0xf>(x);
    x += moved32<ROW_SHR + 4, 0xf>(x);
    return x + moved32<ROW_SHR + 8, 0xf>(x);
}
__device__ __forceinline__ unsigned long long row_scan64(unsigned long long x) {
    x += moved64<ROW_SHR + 1, 0xf>(x);
    x += moved64<ROW_SHR + 2, 0xf>(x);
    x += moved64<ROW_SHR + 4, 0xf>(x);
    return x + moved64<ROW_SHR + 8, 0xf>(x);
}
__device__ __forceinline__ unsigned int wave_scan32(unsigned int x) {
    x = row_scan32(x);
    x += moved32<ROW_BCAST15, 0xa>(x);                   // rows 1 and 3: the last lane of the row before
    return x + moved32<ROW_BCAST31, 0xc>(x);             // rows 2 and 3: lane 31
}
__device__ __forceinline__ unsigned long long wave_scan64(unsigned long long x) {
    x = row_scan64(x);
    x += moved64<ROW_BCAST15, 0xa>(x);
    return x + moved64<ROW_BCAST31, 0xc>(x);
}
template <int LEVEL, bool BYCOUNT>
__device__ __forceinline__ bool scan_level(ScanLds& lds, unsigned long long my_s, unsigned int my_c, HeadState* st, unsigned long long target,
                                           int fix_shift) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    unsigned long long is = wave_scan64(my_s);
    unsigned int ic = wave_scan32(my_c);                 // (a pool holds fewer than 2^31 entries)
    if (lane == 63) { lds.s[wv] = is; lds.c[wv] = ic; }
    __syncthreads();
    {   // the wavefronts before this one: lane i of each row of 16 has wavefront i
        const int i = lane & 15;
        const unsigned long long a = row_scan64(i < wv ? lds.s[i] : 0ull);
        const unsigned int c = row_scan32(i < wv ? lds.c[i] : 0u);
        is += (unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(a >> 32), 15) << 32 | (unsigned int)__builtin_amdgcn_readlane((int)a, 15);
        ic += (unsigned int)__builtin_amdgcn_readlane((int)c, 15);
    }
    __syncthreads();                                     // the caller may scan the next level right away
    const unsigned long long need = (LEVEL == 0) ? target : st->need;
    const unsigned int cexcl = ic - my_c;
    const unsigned long long incl = BYCOUNT ? (unsigned long long)ic : is;
    const unsigned long long excl = BYCOUNT ? (unsigned long long)cexcl : is - my_s;
    if (LEVEL == 0 && t == HIST_BINS - 1 && incl < need) {
        // the whole pool does not reach the target (tau >= 1, or rounding): keep everything
        st->all = 1u;
        return true;
    }
    if (!(excl < need && need <= incl)) return false;
    const int bin = HIST_BINS - 1 - t;
    st->need = need - excl;
    st->cnt_above = (LEVEL == 0 ? 0ull : st->cnt_above) + cexcl;
    st->all = 0u;
    if (LEVEL == 0) st->prefix = ((unsigned)bin) << 20;
    if (LEVEL == 1) st->prefix |= ((unsigned)bin) << 10;
    if (LEVEL == 2) {
        st->prefix |= (unsigned)bin;
        const float theta = __uint_as_float(st->prefix);
        unsigned long long take;
        if (BYCOUNT) {
            take = st->need;                                                 // entries still missing
        } else {
            const unsigned long long each = to_fixed(theta, fix_shift);      // > 0: this bin has mass
            take = (st->need + each - 1) / each;
        }
        if (take > my_c) take = my_c;
        if (take < 1) take = 1;
        st->n_tie = my_c;
        st->take = (unsigned)take;
    }
    return true;
}

// At the last level, when some but not all entries equal to theta are kept: the position of the last kept one, which is all that the mask
// needs to tell them apart.  The entries come out of the candidate list that the second refinement pass left in `cand` (its at most S
// entries share 22 bits with theta); a list that overflowed, or more than TIE_MAX equal entries, leaves TIE_RANKS.
// 12 heads x 112 320 tokens x 288 blocks: the two launches that rank them row by row, another pass over P and a scan of the rows by one
// workgroup per head, took 253 of 3460 us; this end of the last scan adds 9.
constexpr int TIE_MAX = 512;
struct TieLds { HeadState st; unsigned long long last; int n; __align__(16) unsigned int pos[TIE_MAX]; };
__device__ __forceinline__ unsigned long long last_kept_tie(TieLds& lds, const HeadState& st, const unsigned int* __restrict__ p, const int* __restrict__ cand,
                                                            unsigned int n_cand) {
    const int t = threadIdx.x;
    if (t < TIE_MAX) lds.pos[t] = ~0u;                   // after every position
    if (t == 0) { lds.n = 0; lds.last = TIE_RANKS; }
    __syncthreads();
    for (unsigned int i = t; i < n_cand; i += HIST_BINS) {
        const unsigned int pos = (unsigned int)cand[i];
        if (p[pos] == st.prefix) {
            const int at = atomicAdd(&lds.n, 1);         // at most n_tie of them, in any order
            if (at < TIE_MAX) lds.pos[at] = pos;
        }
    }
    __syncthreads();
    if (t < lds.n) {
        const unsigned int mine = lds.pos[t];
        unsigned int before = 0;
        for (int i = 0; i < lds.n; i += 4) {
            const u32x4_t o = *reinterpret_cast<const u32x4_t*>(&lds.pos[i]);
            before += (o.x < mine) + (o.y < mine) + (o.z < mine) + (o.w < mine);
        }
        if (before == st.take - 1u) lds.last = mine;
    }
    __syncthreads();
    return lds.last;
}

template <int LEVEL, bool BYCOUNT>
__global__ __launch_bounds__(HIST_BINS) void scan_level_kernel(const unsigned int* __restrict__ hist_cnt,
                                                               const unsigned long long* __restrict__ hist_sum,
                                                               HeadState* __restrict__ state,
                                                               unsigned long long target, int fix_shift,
                                                               long long pool_size, long long* __restrict__ k_out,
                                                               float* __restrict__ theta_out, const float* __restrict__ P,
                                                               const int* __restrict__ cand, int S) {
    __shared__ ScanLds lds;
    const int bh = blockIdx.x, t = threadIdx.x;
    HeadState st = state[bh];
    if (LEVEL > 0 && st.all) {
        if (LEVEL == 2 && t == 0) { k_out[bh] = pool_size; theta_out[bh] = 0.f; }
        return;
    }
    const long long i = (long long)bh * HIST_BINS + HIST_BINS - 1 - t;
    const unsigned int n_cand = st.n_tie, dropped = st.take;
    const bool mine = scan_level<LEVEL, BYCOUNT>(lds, hist_sum[i], hist_cnt[i], &st, target, fix_shift);
    if (LEVEL < 2) {
        if (mine) state[bh] = st;
        return;
    }
    __shared__ TieLds ties;
    if (t == 0) ties.st.n_tie = ties.st.take = 0u;
    __syncthreads();
    if (mine) ties.st = st;
    __syncthreads();
    st = ties.st;
    if (st.n_tie == 0u) {                                // no bin holds the cut (values that are no numbers)
        if (t == 0) state[bh].n_tie = state[bh].take = 0u;
        return;
    }
    unsigned long long last = TIE_RANKS;
    if (st.take != st.n_tie && !dropped && n_cand <= (unsigned int)S && st.n_tie <= (unsigned int)TIE_MAX)
        last = last_kept_tie(ties, st, reinterpret_cast<const unsigned int*>(P) + bh * pool_size, cand + (long long)bh * S, n_cand);
    if (t == 0) {
        st.need = last;
        state[bh] = st;
        k_out[bh] = (long long)(st.cnt_above + st.take);
        theta_out[bh] = __uint_as_float(st.prefix);
    }
}

// ---------------------------------------------------------------------------------------------
// Pool soft-max mode: "normalised" read as ONE soft-max over the head's whole pool of S * N_b scores.
// With the row soft-max P[q, j] = exp(s_qj - m_q) / d_q already written, the pool value is
//   G[q, j] = exp(s_qj - M) / Z = P[q, j] * w_q,   w_q = d_q exp(m_q - M) / Z,
//   M = max_q m_q,   Z = sum_q d_q exp(m_q - M).
// pool_stat_kernel: one workgroup per head, fixed summation order (double), so Z is reproducible.
__global__ __launch_bounds__(1024) void pool_stat_kernel(const float2* __restrict__ row_stat, float2* __restrict__ pool_stat, int S) {
    __shared__ float sM[1024];
    __shared__ double sZ[1024];
    const int bh = blockIdx.x, t = threadIdx.x;
    const float2* rs = row_stat + (long long)bh * S;
    float m = -INFINITY;
    for (int q = t; q < S; q += 1024) m = fmaxf(m, rs[q].x);
    sM[t] = m;
    __syncthreads();
    for (int off = 512; off >= 1; off >>= 1) {
        if (t < off) sM[t] = fmaxf(sM[t], sM[t + off]);
        __syncthreads();
    }
    const float M = sM[0];
    double z = 0.0;
    for (int q = t; q < S; q += 1024) z += (double)rs[q].y * (double)expf(rs[q].x - M);
    sZ[t] = z;
    __syncthreads();
    for (int off = 512; off >= 1; off >>= 1) {
        if (t < off) sZ[t] += sZ[t + off];
        __syncthreads();
    }
    if (t == 0) pool_stat[bh] = make_float2(M, (float)(1.0 / sZ[0]));
}

// P <- G in place, and the first radix level (count + fixed-point sum per bin) of the new values.
__global__ __launch_bounds__(256) void pool_rescale_kernel(float* __restrict__ P, const float2* __restrict__ row_stat,
                                                           const float2* __restrict__ pool_stat,
                                                           unsigned int* __restrict__ hist_cnt,
                                                           unsigned long long* __restrict__ hist_sum,
                                                           int S, int nb, int fix_shift) {
    __shared__ unsigned int sCnt[HIST_BINS];
    __shared__ unsigned long long sSum[HIST_BINS];
    const int bh = blockIdx.y;
    for (int i = threadIdx.x; i < HIST_BINS; i += 256) { sCnt[i] = 0u; sSum[i] = 0ull; }
    __syncthreads();
    const float2 ps = pool_stat[bh];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int q = blockIdx.x * 4 + wv; q < S; q += gridDim.x * 4) {      // one wavefront per row
        const float2 rs = row_stat[(long long)bh * S + q];
        const float w = rs.y * expf(rs.x - ps.x) * ps.y;
        float* row = P + ((long long)bh * S + q) * nb;
        for (int j = lane; j < nb; j += 64) {
            const float g = row[j] * w;
            row[j] = g;
            const unsigned int bin = min(__float_as_uint(g) >> 20, (unsigned)(HIST_BINS - 1));
            atomicAdd(&sCnt[bin], 1u);
            atomicAdd(&sSum[bin], to_fixed(g, fix_shift));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HIST_BINS; i += 256) {
        const unsigned int c = sCnt[i];
        if (c) {
            atomicAdd(&hist_cnt[(long long)bh * HIST_BINS + i], c);
            atomicAdd(&hist_sum[(long long)bh * HIST_BINS + i], sSum[i]);
        }
    }
}

// Radix levels 1 and 2: histogram of the next 10 bits over the entries whose higher bits
// equal the prefix found so far.  The entries of one bin share every bit above the level's trailing bits (10 at level 1,
// none at level 2), so a bin needs only their number and the sum of those trailing bits: one packed 64-bit LDS atomic
// per candidate (count in bits 40..63), turned into count and fixed-point sum when the workgroup flushes.
// Few, large workgroups (one per compute unit over all heads): every workgroup ends with up to two device-wide atomics per
// bin, and those, not the pass over P, set the time when thousands of workgroups flush.
constexpr int REFINE_NT = 1024;
template <int LEVEL>
__device__ __forceinline__ bool refine_add(unsigned long long* sPk, unsigned int prefix, unsigned int u) {
    constexpr int SHIFT_HI = (LEVEL == 1) ? 20 : 10, SHIFT_LO = (LEVEL == 1) ? 10 : 0;
    if ((u >> SHIFT_HI) != (prefix >> SHIFT_HI)) return false;
    atomicAdd(&sPk[(u >> SHIFT_LO) & (HIST_BINS - 1)], PK_ONE | (unsigned long long)(u & ((1u << SHIFT_LO) - 1u)));
    return true;
}
// count and fixed-point mass of a packed bin
template <int LEVEL>
__device__ __forceinline__ void refine_bin(unsigned long long w, unsigned int prefix, int bin, int fix_shift, unsigned long long& cnt, unsigned long long& sum) {
    constexpr int SHIFT_HI = (LEVEL == 1) ? 20 : 10, SHIFT_LO = (LEVEL == 1) ? 10 : 0;
    cnt = w >> 40;
    // every entry of the bin is (lead | its trailing bits) as a float pattern; to_fixed is linear in the
    // mantissa for a fixed exponent, and the exponent lies in the prefix
    const unsigned int lead = (prefix >> SHIFT_HI << SHIFT_HI) | ((unsigned int)bin << SHIFT_LO);
    const int e = (int)(lead >> 23), sh = e - 150 + fix_shift;
    sum = (cnt && e && sh >= 0) ? (cnt * (unsigned long long)((lead & 0x7fffffu) | 0x800000u) + (w & (PK_ONE - 1))) << sh : 0ull;
}
// The second pass also lists the positions of its candidates, in any order, for the end of the last scan (see last_kept_tie): few, since
// they share 22 bits; REFINE_CAND per workgroup and S per head at most, beyond which they are ranked row by row if need be.
constexpr int REFINE_CAND = 1024;
template <int LEVEL>
__global__ __launch_bounds__(REFINE_NT) void refine_hist_kernel(const float* __restrict__ P, HeadState* __restrict__ state,
                                                          unsigned int* __restrict__ hist_cnt,
                                                          unsigned long long* __restrict__ hist_sum,
                                                          long long pool_size, int fix_shift, int* __restrict__ cand, int S) {
    __shared__ unsigned long long sPk[HIST_BINS];
    __shared__ unsigned int sCand[LEVEL == 2 ? REFINE_CAND : 1], sN, sBase;
    const int bh = blockIdx.y;
    const HeadState st = state[bh];
    if (st.all) return;
    for (int i = threadIdx.x; i < HIST_BINS; i += REFINE_NT) sPk[i] = 0ull;
    if (threadIdx.x == 0) sN = 0u;
    __syncthreads();
    const unsigned int prefix = st.prefix;
    auto take = [&](unsigned int u, long long pos) {     // (a pool holds fewer than 2^31 entries)
        if (refine_add<LEVEL>(sPk, prefix, u) && LEVEL == 2) {
            const unsigned int at = atomicAdd(&sN, 1u);
            if (at < REFINE_CAND) sCand[at] = (unsigned int)pos;
        }
    };
    const u32x4_t* src = reinterpret_cast<const u32x4_t*>(P + (long long)bh * pool_size);
    // 16-byte loads need every head's pool to start on a 16-byte boundary
    const long long n4 = (pool_size % 4 == 0) ? pool_size / 4 : 0;
    // four 16-byte loads in flight per thread: a workgroup takes runs of 4 * REFINE_NT vectors
    for (long long i0 = (long long)blockIdx.x * (4 * REFINE_NT) + threadIdx.x; i0 < n4; i0 += (long long)gridDim.x * (4 * REFINE_NT)) {
        u32x4_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long long i = i0 + REFINE_NT * k;
            const u32x4_t none = {~0u, ~0u, ~0u, ~0u};      // matches no prefix (a NaN pattern; P holds none)
            v[k] = i < n4 ? src[i] : none;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long long e = 4 * (i0 + REFINE_NT * k);
            take(v[k].x, e); take(v[k].y, e + 1); take(v[k].z, e + 2); take(v[k].w, e + 3);
        }
    }
    {
        const unsigned int* s1 = reinterpret_cast<const unsigned int*>(P + (long long)bh * pool_size);
        for (long long i = n4 * 4 + (long long)blockIdx.x * REFINE_NT + threadIdx.x; i < pool_size;
             i += (long long)gridDim.x * REFINE_NT)
            take(s1[i], i);
    }
    __syncthreads();
    if (LEVEL == 2) {
        const unsigned int n = sN;
        if (threadIdx.x == 0 && n) {
            sBase = atomicAdd(&state[bh].n_tie, min(n, (unsigned int)REFINE_CAND));
            if (n > REFINE_CAND) atomicOr(&state[bh].take, 1u);
        }
        __syncthreads();
        const unsigned int base = n ? sBase : 0u;
        for (unsigned int i = threadIdx.x; i < min(n, (unsigned int)REFINE_CAND) && base + i < (unsigned int)S; i += REFINE_NT)
            cand[(long long)bh * S + base + i] = (int)sCand[i];
    }
    for (int i = threadIdx.x; i < HIST_BINS; i += REFINE_NT) {
        unsigned long long cnt, sum;
        refine_bin<LEVEL>(sPk[i], prefix, i, fix_shift, cnt, sum);
        if (cnt) {
            atomicAdd(&hist_cnt[(long long)bh * HIST_BINS + i], (unsigned int)cnt);
            if (sum) atomicAdd(&hist_sum[(long long)bh * HIST_BINS + i], sum);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Per-row count of entries equal to theta.  Only needed when some but not all of them belong
// to the top k and they are too many for last_kept_tie; otherwise the kernel returns at once.
__global__ __launch_bounds__(256) void tie_count_kernel(const float* __restrict__ P, const HeadState* __restrict__ state,
                                                        int* __restrict__ ties, int S, int nb) {
    const int bh = blockIdx.y;
    const HeadState st = state[bh];
    if (st.all || st.take == st.n_tie || st.need != TIE_RANKS) return;
    const int lane = threadIdx.x & 63;
    const int gw = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int n_gw = gridDim.x * 4;
    for (int q = gw; q < S; q += n_gw) {
        const unsigned int* row = reinterpret_cast<const unsigned int*>(P + ((long long)bh * S + q) * nb);
        int c = 0;
        for (int j0 = 0; j0 < nb; j0 += 64) {
            int j = j0 + lane;
            bool tie = (j < nb) && (row[j] == st.prefix);
            c += __popcll(__ballot(tie));
        }
        if (lane == 0) ties[(long long)bh * S + q] = c;
    }
}

// Exclusive prefix sum of in[bh][0..S) into out[bh][0..S], out[bh][S] = total.  One workgroup
// per head; a no-op for heads that do not need tie ranks.
__global__ __launch_bounds__(SCAN_THREADS) void row_scan_kernel(const int* __restrict__ in, int* __restrict__ out,
                                                                const HeadState* __restrict__ state, int S) {
    __shared__ int sW[SCAN_THREADS / 64];
    __shared__ int sCarry;
    // a batch of SCAN_THREADS * SCAN_ITEMS values passes through LDS so that global memory is read and written in whole
    // rows of consecutive lanes while every thread scans SCAN_ITEMS consecutive values; item i sits at i + i / SCAN_ITEMS
    // (a thread's items then start SCAN_ITEMS + 1 words apart: no bank conflicts)
    __shared__ int sBuf[SCAN_THREADS * (SCAN_ITEMS + 1)];
    const int bh = blockIdx.x, t = threadIdx.x;
    const HeadState st = state[bh];
    if (st.all || st.take == st.n_tie || st.need != TIE_RANKS) return;
    const int* src = in + (long long)bh * S;
    int* dst = out + (long long)bh * (S + 1);
    if (t == 0) sCarry = 0;
    __syncthreads();
    for (int base = 0; base < S; base += SCAN_THREADS * SCAN_ITEMS) {
#pragma unroll
        for (int e = 0; e < SCAN_ITEMS; ++e) {
            const int li = e * SCAN_THREADS + t;
            sBuf[li + li / SCAN_ITEMS] = (base + li < S) ? src[base + li] : 0;
        }
        __syncthreads();
        int v[SCAN_ITEMS];
        int sum = 0;
#pragma unroll
        for (int e = 0; e < SCAN_ITEMS; ++e) {
            v[e] = sBuf[t * (SCAN_ITEMS + 1) + e];
            sum += v[e];
        }
        // inclusive scan of `sum` across the workgroup: wave scan, then scan of wave totals
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            int n = __shfl_up(incl, off, 64);
            if ((t & 63) >= off) incl += n;
        }
        if ((t & 63) == 63) sW[t >> 6] = incl;
        __syncthreads();
        int wave_base = 0;
        for (int w = 0; w < (t >> 6); ++w) wave_base += sW[w];
        int run = sCarry + wave_base + incl - sum;
#pragma unroll
        for (int e = 0; e < SCAN_ITEMS; ++e) {
            sBuf[t * (SCAN_ITEMS + 1) + e] = run;
            run += v[e];
        }
        __syncthreads();
        if (t == SCAN_THREADS - 1) sCarry = run;
#pragma unroll
        for (int e = 0; e < SCAN_ITEMS; ++e) {
            const int li = e * SCAN_THREADS + t;
            if (base + li < S) dst[base + li] = sBuf[li + li / SCAN_ITEMS];
        }
        __syncthreads();
    }
    if (t == 0) dst[S] = sCarry;
}

// ---------------------------------------------------------------------------------------------
// TopkMask (Eq. 3): bit (q, j) = P[q, j] is among the k best of the head.  One wavefront per
// 64 consecutive queries.  Also counts, per wavefront, how many of its queries keep each block
// (the raw material of the block-major list).
// Block that holds block-order position q (blk_off ascending, blk_off[0] = 0, blk_off[nb] = S).
__device__ __forceinline__ int block_of_position(const int* __restrict__ blk_off, int nb, int q) {
    int lo = 0, hi = nb;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (blk_off[mid] <= q) lo = mid; else hi = mid;
    }
    return lo;
}

// Workgroup i of n runs on XCD i % 8; this index makes the workgroups of one XCD neighbours in the work list, so runs
// that different workgroups write into the same cache line meet in one L2.
__device__ __forceinline__ int xcd_contiguous(int i, int n) {
    const int per = n / 8;
    return i < per * 8 ? (i % 8) * per + i / 8 : i;
}

// One mask word per lane (lane = row of the wavefront's 64 queries; blocks 32 wd to 32 wd + jn - 1): how many of the rows keep each block, to
// wcnt[block][w].  Returns the sum.
__device__ __forceinline__ int count_word(unsigned int word, int wd, int jn, int* __restrict__ wcnt, long long bh_nb, int n_waves, int w) {
    const int lane = threadIdx.x & 63;
    int kept = 0, mine = 0;                      // lane b: the count of block 32 wd + b, so that all of them leave in one store
    for (int bit = 0; bit < jn; ++bit) {
        const int c = __popcll(__ballot((word >> bit) & 1u));
        kept += c;
        mine = lane == bit ? c : mine;
    }
    if (lane < jn) wcnt[(bh_nb + wd * 32 + lane) * n_waves + w] = mine;
    return kept;
}

// Mask of 64 rows of P by one wavefront (its LDS instructions execute in order: no barriers).  tie_base: per row of the head, entries equal
// to theta in the rows before, used for TIE_RANKS.  own_blk_off: null, or blk_off when every query also keeps the block it lies in
// itself; query_pos: null when query q sits at block-order position q, else the position of every query (queries kept in the caller's
// token order).
// Bound by the read of P.  The rows are one contiguous run of values, read flat with 16 loads in flight; a comparison of 64 of them is 64
// bits of one flat mask in the LDS, from which a row's words are cut with two reads and a shift.  Neighbouring workgroups, whose counts
// share cache lines, run on one XCD.  12 heads: 32 760 x 84 blocks 38.1 -> 29.2 us, 112 320 x 288, 1.7 GB, 375 -> 354 (375 without the
// order of the workgroups); 32 x 6601 x 36 13.7 -> 10.9.  Before: 16-byte loads, the bits set by LDS atomics.
constexpr int MASK_LOADS = 16;
__global__ __launch_bounds__(256) void mask_kernel(const float* __restrict__ P, const HeadState* __restrict__ state,
                                                   const int* __restrict__ tie_base, unsigned int* __restrict__ mask,
                                                   int* __restrict__ wtot, int* __restrict__ wcnt,
                                                   int S, int nb, int n_waves, const int* __restrict__ own_blk_off,
                                                   const int* __restrict__ query_pos) {
    __shared__ unsigned long long sBits[4][VMOBA_MAX_BLOCKS + 1];
    const int bh = blockIdx.y, lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = xcd_contiguous(blockIdx.x, gridDim.x) * 4 + wv;
    if (w >= n_waves) return;
    const HeadState st = state[bh];
    unsigned long long* bits = sBits[wv];
    const int q0 = w * 64, words = (nb + 31) / 32, rows = min(64, S - q0), n_el = rows * nb;
    const unsigned int* tile = reinterpret_cast<const unsigned int*>(P + ((long long)bh * S + q0) * nb);
    // entries equal to theta: all kept, kept up to a position of the head's pool (last_kept_tie), or (rare) kept by rank
    const bool whole = st.all || st.take == st.n_tie, ranked = !whole && st.need == TIE_RANKS;
    const unsigned int least = st.all ? 0u : st.prefix + (whole ? 0u : 1u);
    const long long last_tie = whole || ranked ? -1 : (long long)st.need - (long long)q0 * nb;      // in this tile
    unsigned int rank = ranked ? (unsigned int)tie_base[(long long)bh * (S + 1) + q0] : 0u;
    auto chunk = [&](int e0, auto full) {
        unsigned int x[MASK_LOADS];
#pragma unroll
        for (int u = 0; u < MASK_LOADS; ++u) {
            const int e = e0 + u * 64 + lane;
            x[u] = decltype(full)::value || e < n_el ? tile[e] : 0u;
        }
#pragma unroll
        for (int u = 0; u < MASK_LOADS; ++u) {
            if (!decltype(full)::value && e0 + u * 64 >= n_el) break;
            unsigned long long keep = __ballot(x[u] >= least);          // (no row's words hold a bit past the run)
            if (!whole) {
                const unsigned long long tie = __ballot(x[u] == st.prefix);
                if (tie) {
                    const unsigned int before = __popcll(tie & ((1ull << lane) - 1ull));
                    const bool in = ranked ? rank + before < st.take : e0 + u * 64 + lane <= last_tie;
                    keep |= tie & __ballot(in);
                    rank += __popcll(tie);
                }
            }
            if (lane == 0) bits[(e0 >> 6) + u] = keep;
        }
    };
    int e0 = 0;
    for (; e0 + 64 * MASK_LOADS <= n_el; e0 += 64 * MASK_LOADS) chunk(e0, std::true_type{});
    if (e0 < n_el) chunk(e0, std::false_type{});
    asm volatile("" ::: "memory");
    // lane = row
    const int q = q0 + lane;
    const bool live = lane < rows;
    const int own = own_blk_off && live ? block_of_position(own_blk_off, nb, query_pos ? query_pos[q] : q) : -1;
    int kept = 0;
    for (int wd = 0; wd < words; ++wd) {
        const int jn = min(32, nb - wd * 32);
        unsigned int g = 0u;
        if (live) {
            const int at = lane * nb + wd * 32, sh = at & 63;
            g = (unsigned int)(bits[at >> 6] >> sh | bits[(at >> 6) + 1] << 1 << (63 - sh)) & (~0u >> (32 - jn));
            if (wd == (own >> 5)) g |= 1u << (own & 31);       // own = -1: no word matches
            mask[((long long)bh * S + q) * words + wd] = g;
        }
        kept += count_word(g, wd, jn, wcnt, (long long)bh * nb, n_waves, w);
    }
    if (lane == 0) wtot[(long long)bh * n_waves + w] = kept;
}

// Common end of the per-query selections: lane = row of the wavefront's 64 queries, sKeep[row] its mask words.  Adds the
// query's own block, writes the mask and counts, per wavefront, how many of its queries keep each block (as mask_kernel does).
__device__ __forceinline__ void store_local_mask(const unsigned int (*sKeep)[VMOBA_MAX_MASK_WORDS + 1], unsigned int* __restrict__ mask,
                                                 int* __restrict__ wtot, int* __restrict__ wcnt, int bh, int w, int q0, int rows, bool active,
                                                 int S, int nb, int n_waves, const int* __restrict__ own_blk_off, const int* __restrict__ query_pos) {
    const int lane = threadIdx.x & 63, words = (nb + 31) / 32;
    const int q = q0 + lane;
    const bool live = lane < rows;
    const int own = (own_blk_off && live) ? block_of_position(own_blk_off, nb, query_pos ? query_pos[q] : q) : -1;
    if (!active) return;
    int kept = 0;
    for (int wd = 0; wd < words; ++wd) {
        unsigned int g = 0;
        if (live) {
            g = sKeep[lane][wd];
            if (wd == (own >> 5)) g |= 1u << (own & 31);
            mask[((long long)bh * S + q) * words + wd] = g;
        }
        kept += count_word(g, wd, min(32, nb - wd * 32), wcnt, (long long)bh * nb, n_waves, w);
    }
    if (lane == 0) wtot[(long long)bh * n_waves + w] = kept;
}

// Per-query ("local") selection, the block-choice variants of the paper's ablation and of its training-free runs.
//
// Top-k: a query keeps its `topk` most similar blocks, equal values by lowest block index.  One wavefront per 64 queries;
// a row is held by 1 << lpr_log2 lanes, CPL columns each, in registers, and the k-th largest value is found bit by bit
// (soft-max values are not negative: their bits order like integers): two instructions per column and bit, and rows whose
// count hits k before the last bit are done -- usually after about half of the 30 bits.
// Bound by these instructions and by reading P.  720p, 12 heads, 40 blocks, k = 10: 1079 -> 74 us (before: a row spread over the
// lanes, every lane counting what ranks before its own columns -- nb LDS broadcasts and two barriers for every row, its loads
// waited for); the whole selection with 288 blocks, k = 60, 56 160 tokens: 11.0 -> 1.65 ms.
// A row of NaNs keeps every block (the list capacity then reports the head).
template <int CPL>
__global__ __launch_bounds__(256, 4) void local_topk_kernel(const float* __restrict__ P, unsigned int* __restrict__ mask,
                                                         int* __restrict__ wtot, int* __restrict__ wcnt, int S, int nb, int n_waves, int topk,
                                                         int lpr_log2, const int* __restrict__ own_blk_off, const int* __restrict__ query_pos) {
    __shared__ unsigned int sKeep[4][64][VMOBA_MAX_MASK_WORDS + 1];
    const int bh = blockIdx.y;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int w = blockIdx.x * 4 + wv;
    const bool active = w < n_waves;
    const int q0 = active ? w * 64 : 0;
    const int rows = active ? min(64, S - q0) : 0;
    const int k = min(topk, nb);
    const int lpr = 1 << lpr_log2, part = lane & (lpr - 1), c0 = part * CPL;
    const bool aligned = (nb & 3) == 0 && (reinterpret_cast<uintptr_t>(P) & 15) == 0;          // rows start 16-byte aligned
    for (int wd = 0; wd < (nb + 31) / 32; ++wd) sKeep[wv][lane][wd] = 0u;
    auto sum_row = [&](int v) {                  // over the lanes of a row
        for (int off = 1; off < lpr; off <<= 1) v += __shfl_xor(v, off, 64);
        return v;
    };
    for (int batch = 0; batch < lpr; ++batch) {
        const int r = (batch << (6 - lpr_log2)) + (lane >> lpr_log2);
        const bool live = r < rows;
        const unsigned int* row = reinterpret_cast<const unsigned int*>(P) + ((long long)bh * S + q0 + (live ? r : 0)) * nb + c0;
        unsigned int v[CPL];                     // columns past the row's end: 0, below every candidate and after every other 0
        if (aligned) {
#pragma unroll
            for (int i = 0; i < CPL; i += 4) {
                u32x4_t x = {0u, 0u, 0u, 0u};
                if (live && c0 + i < nb) x = *reinterpret_cast<const u32x4_t*>(row + i);
                v[i] = x.x; v[i + 1] = x.y; v[i + 2] = x.z; v[i + 3] = x.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < CPL; ++i) v[i] = (live && c0 + i < nb) ? row[i] : 0u;
        }
        unsigned int top = v[0];
#pragma unroll
        for (int i = 1; i < CPL; ++i) top = max(top, v[i]);
        for (int off = 1; off < lpr; off <<= 1) top = max(top, (unsigned int)__shfl_xor((int)top, off, 64));
        // kth: count(v >= kth) >= k; done: the count is k (or every column is kept)
        unsigned int kth = 0;
        bool done = !live || k == nb || top > 0x7f800000u;
        for (int bit = 29; bit >= 0 && __ballot(!done); --bit) {             // values below 2 have 30 significant bits
            const unsigned int cand = kth | (1u << bit);
            int n = 0;
#pragma unroll
            for (int i = 0; i < CPL; ++i) n += v[i] >= cand ? 1 : 0;
            n = sum_row(n);
            if (!done && n >= k) {
                kth = cand;
                done = n == k;
            }
        }
        // more than k columns reach the k-th value only where several equal it: of these, the first ones
        int take = 64 * 512;                     // columns v > kth are kept, and the first `take` of v == kth
        if (__ballot(!done)) {
            int n_gt = 0, n_eq = 0;
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                n_gt += v[i] > kth ? 1 : 0;
                n_eq += v[i] == kth ? 1 : 0;
            }
            n_gt = sum_row(n_gt);
            int before = n_eq;                   // equal columns in the row's lanes up to this one
            for (int off = 1; off < lpr; off <<= 1) {
                const int o = __shfl_up(before, off, 64);
                if (part >= off) before += o;
            }
            if (!done) take = k - n_gt - (before - n_eq);
        }
        unsigned long long keep = 0;
        if (__ballot(!done)) {
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const bool eq = v[i] == kth;
                keep |= v[i] > kth || (eq && take > 0) ? 1ull << i : 0ull;
                take -= eq ? 1 : 0;
            }
        } else {
#pragma unroll
            for (int i = 0; i < CPL; ++i) keep |= v[i] >= kth ? 1ull << i : 0ull;
        }
        if (c0 + CPL > nb) keep &= nb > c0 ? (1ull << (nb - c0)) - 1ull : 0ull;
        if (live) {
            const int wd = c0 >> 5, sh = c0 & 31;
            const unsigned int w0 = (unsigned int)(keep << sh), w1 = (unsigned int)((keep << sh) >> 32);
            const unsigned int w2 = sh ? (unsigned int)(keep >> (64 - sh)) : 0u;
            if (w0) atomicOr(&sKeep[wv][r][wd], w0);
            if (w1) atomicOr(&sKeep[wv][r][wd + 1], w1);
            if (w2) atomicOr(&sKeep[wv][r][wd + 2], w2);
        }
    }
    __syncthreads();
    store_local_mask(sKeep[wv], mask, wtot, wcnt, bh, w, q0, rows, active, S, nb, n_waves, own_blk_off, query_pos);
}

// Threshold: a query keeps the shortest descending prefix of its own row whose sum reaches tau; entry j' ranks before j when
// it is larger, or equal with a lower block index.  One wavefront per 64 queries; a row is spread over the lanes (NCOL columns
// each) and every lane sums, in column order, what ranks before its own entries.  Bound by these instructions, nb * NCOL times
// three per row: soft-max values are not negative, so their bits compare like integers and "larger, or equal with a lower
// index" is one comparison, with the value minus one bit for columns that come later.  The next row's values are fetched
// while a row is worked on, and a wavefront's LDS row is its own: no barriers.  The whole selection at 480p, 12 heads, 84 blocks:
// 1.36 -> 0.62 ms (with barriers, every row's loads waited for and twice the instructions before).
// A row of NaNs keeps every block.
template <int NCOL>
__global__ __launch_bounds__(256) void local_threshold_kernel(const float* __restrict__ P, unsigned int* __restrict__ mask,
                                                              int* __restrict__ wtot, int* __restrict__ wcnt,
                                                              int S, int nb, int n_waves, float tau,
                                                              const int* __restrict__ own_blk_off, const int* __restrict__ query_pos) {
    __shared__ __align__(16) int sRow[4][NCOL * 64];
    __shared__ unsigned int sKeep[4][64][VMOBA_MAX_MASK_WORDS + 1];
    const int bh = blockIdx.y;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int w = blockIdx.x * 4 + wv;
    const bool active = w < n_waves;
    const int q0 = active ? w * 64 : 0;
    const int rows = active ? min(64, S - q0) : 0;
    const int* base = reinterpret_cast<const int*>(P) + ((long long)bh * S + q0) * nb;
    int* const sr = sRow[wv];
    int nx[NCOL];
    auto fetch = [&](int r) {
#pragma unroll
        for (int c = 0; c < NCOL; ++c) nx[c] = c * 64 + lane < nb ? base[(long long)r * nb + c * 64 + lane] : -1;     // -1: before nothing
    };
    if (rows > 0) fetch(0);
    for (int r = 0; r < rows; ++r) {
        int v[NCOL];
        bool nan = false;
#pragma unroll
        for (int c = 0; c < NCOL; ++c) {
            v[c] = nx[c];
            sr[c * 64 + lane] = v[c];
            nan |= c * 64 + lane < nb && __int_as_float(v[c]) != __int_as_float(v[c]);
        }
        const bool all = tau >= 1.f || __ballot(nan);
        asm volatile("" ::: "memory");                       // a wavefront's LDS instructions execute in order
        if (r + 1 < rows) fetch(r + 1);
        float before[NCOL];
#pragma unroll
        for (int c = 0; c < NCOL; ++c) before[c] = 0.f;
        if (!all) {
#pragma unroll
            for (int cp = 0; cp < NCOL; ++cp) {
                const int n4 = min(64, nb - cp * 64);
                for (int jp = 0; jp < n4; jp += 4) {
                    const u32x4_t x4 = *reinterpret_cast<const u32x4_t*>(sr + cp * 64 + jp);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int x = (int)x4[u];
#pragma unroll
                        for (int c = 0; c < NCOL; ++c) {
                            const int later = cp < c ? 1 : cp > c ? 0 : (jp + u < lane ? 1 : 0);     // column jp + u comes before this lane's
                            before[c] += x > v[c] - later ? __int_as_float(x) : 0.f;
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NCOL; ++c) {
            const unsigned long long bal = __ballot(c * 64 + lane < nb && (all || before[c] < tau));
            if (lane == 0) {
                sKeep[wv][r][2 * c] = (unsigned)bal;
                sKeep[wv][r][2 * c + 1] = (unsigned)(bal >> 32);
            }
        }
        asm volatile("" ::: "memory");
    }
    __syncthreads();
    store_local_mask(sKeep[wv], mask, wtot, wcnt, bh, w, q0, rows, active, S, nb, n_waves, own_blk_off, query_pos);
}

// Offsets of both list forms, in two small launches.
// wave_scan_kernel, one workgroup per (row, head), rows 0..nb:
//  * row j < nb: wcnt[j][w] (pairs of block j among the 64 queries of wavefront w) -> its exclusive scan over w, in place:
//    where wavefront w's entries of block j start inside the block's list; the total is the block's count;
//  * row nb: wtot[w] (pairs kept by the 64 queries of wavefront w) -> its exclusive scan, in place: where their rows
//    start in the query-major lists; the total is row_ptr[S].
__global__ __launch_bounds__(256) void wave_scan_kernel(int* __restrict__ wcnt, int* __restrict__ wtot,
                                                        int* __restrict__ row_tot, int nb, int n_waves) {
    __shared__ int sW[4];
    __shared__ int sCarry;
    const int j = blockIdx.x, bh = blockIdx.y, t = threadIdx.x;
    int* col = j < nb ? wcnt + ((long long)bh * nb + j) * n_waves : wtot + (long long)bh * n_waves;
    if (t == 0) sCarry = 0;
    __syncthreads();
    for (int base = 0; base < n_waves; base += 256) {
        const int i = base + t;
        const int v = (i < n_waves) ? col[i] : 0;
        int incl = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            int n = __shfl_up(incl, off, 64);
            if ((t & 63) >= off) incl += n;
        }
        if ((t & 63) == 63) sW[t >> 6] = incl;
        __syncthreads();
        int wave_base = 0;
        for (int w = 0; w < (t >> 6); ++w) wave_base += sW[w];
        const int excl = sCarry + wave_base + incl - v;
        if (i < n_waves) col[i] = excl;
        __syncthreads();
        if (t == 255) sCarry = excl + v;
        __syncthreads();
    }
    if (t == 0) row_tot[(long long)bh * (nb + 1) + j] = sCarry;
}

// blk_ptr = exclusive scan of the block counts, with the capacity check.  One wavefront per head, a run of blocks per
// lane.  A head that kept more than `cap` pairs gets an all-zero blk_ptr -- to the attention calls it selected nothing,
// so no list entry of it is ever read (the merge kernels recognise the same head by row_ptr[S] > cap) -- and the status
// word is set.  Also row_ptr[S], the head's number of pairs; write_k != 0 (per-query modes, or every query keeps its
// own block: the number of kept pairs is not the k of the cut) copies it to k_out, write_k == 2 also clears theta_out.
__device__ __forceinline__ void block_offsets(const int* cnt, int* __restrict__ blk_ptr, int* __restrict__ row_ptr, long long* __restrict__ k_out,
                                              float* __restrict__ theta_out, int bh, int nb, int S, long long cap, int* __restrict__ dev_status,
                                              int write_k) {
    const int lane = threadIdx.x & 63;
    const int per = (nb + 63) / 64;                  // consecutive blocks per lane
    const int j0 = min(nb, lane * per), j1 = min(nb, j0 + per);
    int* out = blk_ptr + (long long)bh * (nb + 1);
    int mine = 0;
    for (int j = j0; j < j1; ++j) mine += cnt[j];
    int incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    const long long total = __shfl(incl, 63, 64);
    const bool fits = total <= cap;
    int run = incl - mine;
    for (int j = j0; j < j1; ++j) {
        out[j] = fits ? run : 0;
        run += cnt[j];
    }
    if (lane == 0) {
        out[nb] = fits ? (int)total : 0;
        if (!fits) atomicExch(dev_status, (int)VMOBA_ERR_CAPACITY);
        row_ptr[(long long)bh * (S + 1) + S] = cnt[nb];
        if (write_k) k_out[bh] = cnt[nb];
        if (write_k == 2) theta_out[bh] = 0.f;
    }
}

__global__ __launch_bounds__(64) void blk_ptr_kernel(const int* __restrict__ row_tot, int* __restrict__ blk_ptr,
                                                     int* __restrict__ row_ptr, long long* __restrict__ k_out,
                                                     float* __restrict__ theta_out, int nb, int S, long long cap,
                                                     int* __restrict__ dev_status, int write_k) {
    block_offsets(row_tot + (long long)blockIdx.x * (nb + 1), blk_ptr, row_ptr, k_out, theta_out, blockIdx.x, nb, S, cap, dev_status, write_k);
}

// Offsets of both list forms for one head by the 16 wavefronts of a workgroup (what wave_scan_kernel and blk_ptr_kernel do).
__device__ __forceinline__ void head_offsets(int* sTot, int* __restrict__ wcnt, int* __restrict__ wtot, int* __restrict__ blk_ptr, int* __restrict__ row_ptr,
                                             long long* __restrict__ k_out, float* __restrict__ theta_out, int bh, int nb, int S, int n_waves, long long cap,
                                             int* __restrict__ dev_status, int write_k) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int j = wv; j <= nb; j += 16) {
        int* col = j < nb ? wcnt + ((long long)bh * nb + j) * n_waves : wtot + (long long)bh * n_waves;
        int carry = 0;
        for (int base = 0; base < n_waves; base += 64) {
            const int v = base + lane < n_waves ? col[base + lane] : 0;
            int incl = v;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(incl, off, 64);
                if (lane >= off) incl += o;
            }
            if (base + lane < n_waves) col[base + lane] = carry + incl - v;
            carry += __shfl(incl, 63, 64);
        }
        if (lane == 0) sTot[j] = carry;
    }
    __syncthreads();
    if (wv == 0) block_offsets(sTot, blk_ptr, row_ptr, k_out, theta_out, bh, nb, S, cap, dev_status, write_k);
}

// Everything between the scores and the lists -- the three radix levels, tie ranks, mask, list offsets -- for a small pool, one
// workgroup per head in one launch instead of ten that take 2 to 7 us each whatever their size.  Bound by the instructions of one compute
// unit and a dozen barriers.  A head's values are read once, beside the histogram, and stay in registers for both refinement levels
// and the mask (32 of the 128 a thread of 1024 may have).  The mask is first one flat run of bits, a comparison per 64 values; a
// row's words are cut out of it with two reads and a shift.  Same integers, same results as the kernels above.
// 12 heads x 1560 tokens x 20 blocks: 23.1 -> 16.7 us, 2 heads x 512 x 16: 15.9 -> 9.4 (before: values fetched for every pass, mask bits by
// LDS atomics, scans by shuffles); with the values kept but the bits still by atomics 22.3 and 14.0.  The line lies at 2^15 values: before,
// the separate launches were as fast from about 6 x 10^4 on, and more values would not fit the registers.
constexpr long long SMALL_POOL = 1 << 15;
constexpr int SMALL_ROWS = 4096, SMALL_WORDS = 4;
constexpr int SMALL_VALS = (int)(SMALL_POOL / HIST_BINS);
// (blocks + 1) * (groups of 64 queries) <= pool / 64 + blocks + groups + 1
constexpr int SMALL_COUNTS = 1024;
static_assert(SMALL_POOL / 64 + SMALL_WORDS * 32 + SMALL_ROWS / 64 + 1 <= SMALL_COUNTS, "counts of a head must fit the LDS array");
template <bool BYCOUNT>
__global__ __launch_bounds__(HIST_BINS) void small_cut_kernel(const float* __restrict__ P, const unsigned int* __restrict__ hist_cnt,
                                                              const unsigned long long* __restrict__ hist_sum, unsigned long long target, int fix_shift,
                                                              unsigned int* __restrict__ mask, int* __restrict__ wtot, int* __restrict__ wcnt,
                                                              int* __restrict__ blk_ptr, int* __restrict__ row_ptr, long long* __restrict__ k_out,
                                                              float* __restrict__ theta_out, int* __restrict__ dev_status, int S, int nb, int n_waves,
                                                              long long cap, const int* __restrict__ own_blk_off, const int* __restrict__ query_pos,
                                                              int write_k) {
    constexpr int NW = HIST_BINS / 64;
    __shared__ ScanLds scan;
    __shared__ HeadState sState;
    __shared__ unsigned long long sPk[HIST_BINS];
    __shared__ unsigned long long sKeep[SMALL_POOL / 64 + 1], sTie[SMALL_POOL / 64];   // a bit per value: kept, equal to theta
    __shared__ int sCnt[SMALL_COUNTS];                           // [block, then all blocks][group of 64 queries]
    __shared__ int sTot[SMALL_WORDS * 32 + 1];
    __shared__ int sW[NW];
    const int bh = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int pool = S * nb, words = (nb + 31) / 32;
    const unsigned int* p = reinterpret_cast<const unsigned int*>(P) + (long long)bh * pool;
    // ---- the head's values: value t + 1024 k in v[k]
    const long long hi = (long long)bh * HIST_BINS + HIST_BINS - 1 - t;
    const unsigned long long h_sum = hist_sum[hi];
    const unsigned int h_cnt = hist_cnt[hi];
    unsigned int v[SMALL_VALS];
#pragma unroll
    for (int k = 0; k < SMALL_VALS; ++k) {
        const int e = t + k * HIST_BINS;
        v[k] = ~0u;                                      // matches no prefix
        if (e < pool) v[k] = p[e];
    }
    sPk[t] = 0ull;
    // ---- the cut
    HeadState st = {0, 0, 0, 0, 0, 0};
    if (t == 0) sState = st;
    __syncthreads();
    if (scan_level<0, BYCOUNT>(scan, h_sum, h_cnt, &st, target, fix_shift)) sState = st;
    __syncthreads();
    st = sState;
    auto refine = [&](auto level) {
        constexpr int LEVEL = decltype(level)::value;
#pragma unroll
        for (int k0 = 0; k0 < SMALL_VALS; k0 += 4)
            if (k0 * HIST_BINS < pool)
#pragma unroll
                for (int k = k0; k < k0 + 4; ++k) refine_add<LEVEL>(sPk, st.prefix, v[k]);
        __syncthreads();
        const int bin = HIST_BINS - 1 - t;
        unsigned long long cnt, sum;
        refine_bin<LEVEL>(sPk[bin], st.prefix, bin, fix_shift, cnt, sum);
        sPk[bin] = 0ull;                                 // for the next level; the scan's barriers lie between
        if (scan_level<LEVEL, BYCOUNT>(scan, sum, (unsigned int)cnt, &st, target, fix_shift)) sState = st;
        __syncthreads();
        st = sState;
    };
    if (!st.all) {                                       // same decision in every thread
        refine(std::integral_constant<int, 1>{});
        refine(std::integral_constant<int, 2>{});
    }
    if (t == 0) {
        k_out[bh] = st.all ? (long long)pool : (long long)(st.cnt_above + st.take);
        theta_out[bh] = st.all ? 0.f : __uint_as_float(st.prefix);
    }
    // ---- mask bits; of entries equal to theta the first `take`
    const bool all_ties = st.all || st.take == st.n_tie;
    const unsigned int least = st.all ? 0u : st.prefix + (all_ties ? 0u : 1u);
#pragma unroll
    for (int k0 = 0; k0 < SMALL_VALS; k0 += 4) {
        if (k0 * HIST_BINS < pool) {
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) {          // (no row's words hold a bit past the pool)
                const unsigned long long keep = __ballot(v[k] >= least), tie = __ballot(v[k] == st.prefix);
                if (lane == 0) { sKeep[k * NW + wv] = keep; sTie[k * NW + wv] = tie; }
            }
        }
    }
    __syncthreads();
    if (!all_ties) {
        const int n_words = (pool + 63) / 64;            // at most 512: one per thread
        unsigned long long tie = t < n_words ? sTie[t] : 0ull;
        const unsigned int incl = wave_scan32((unsigned int)__popcll(tie));
        if (lane == 63) sW[wv] = (int)incl;
        __syncthreads();
        unsigned int before = incl - (unsigned int)__popcll(tie);
        for (int w = 0; w < wv; ++w) before += (unsigned int)sW[w];
        unsigned long long keep = 0ull;
        for (; tie && before < st.take; ++before) {
            const unsigned long long low = tie & (0ull - tie);
            keep |= low;
            tie ^= low;
        }
        if (keep) sKeep[t] |= keep;
        __syncthreads();
    }
    // ---- mask words and the counts per block and group of 64 queries (lane = row)
    for (int w = wv; w < n_waves; w += NW) {
        const int q = w * 64 + lane;
        const bool live = q < S;
        const int own = own_blk_off && live ? block_of_position(own_blk_off, nb, query_pos ? query_pos[q] : q) : -1;
        const unsigned int* flat = reinterpret_cast<const unsigned int*>(sKeep);
        int kept = 0;
        for (int wd = 0; wd < words; ++wd) {
            const int jn = min(32, nb - wd * 32);
            unsigned int g = 0u;
            if (live) {
                const int at = q * nb + wd * 32;
                const unsigned long long two = (unsigned long long)flat[(at >> 5) + 1] << 32 | flat[at >> 5];
                g = (unsigned int)(two >> (at & 31)) & (~0u >> (32 - jn));
                if (wd == (own >> 5)) g |= 1u << (own & 31);           // own = -1: no word matches
                mask[((long long)bh * S + q) * words + wd] = g;
            }
            int mine = 0;                                              // lane b: the count of block 32 wd + b
            for (int bit = 0; bit < jn; ++bit) {
                const int c = __popcll(__ballot((g >> bit) & 1u));
                kept += c;
                mine = lane == bit ? c : mine;
            }
            if (lane < jn) sCnt[(wd * 32 + lane) * n_waves + w] = mine;
        }
        if (lane == 0) sCnt[nb * n_waves + w] = kept;
    }
    __syncthreads();
    // ---- list offsets (what wave_scan_kernel and blk_ptr_kernel do); at most 64 groups of queries
    for (int j = wv; j <= nb; j += NW) {
        const int c = lane < n_waves ? sCnt[j * n_waves + lane] : 0;
        const int incl = (int)wave_scan32((unsigned int)c);
        int* col = j < nb ? wcnt + ((long long)bh * nb + j) * n_waves : wtot + (long long)bh * n_waves;
        if (lane < n_waves) col[lane] = incl - c;
        if (lane == 63) sTot[j] = incl;
    }
    __syncthreads();
    if (wv == 0) block_offsets(sTot, blk_ptr, row_ptr, k_out, theta_out, bh, nb, S, cap, dev_status, write_k);
}

__global__ __launch_bounds__(1024) void head_offsets_kernel(int* __restrict__ wcnt, int* __restrict__ wtot, int* __restrict__ blk_ptr,
                                                            int* __restrict__ row_ptr, long long* __restrict__ k_out, float* __restrict__ theta_out,
                                                            int nb, int S, int n_waves, long long cap, int* __restrict__ dev_status, int write_k) {
    __shared__ int sTot[VMOBA_MAX_BLOCKS + 1];
    head_offsets(sTot, wcnt, wtot, blk_ptr, row_ptr, k_out, theta_out, blockIdx.x, nb, S, n_waves, cap, dev_status, write_k);
}

// Fill q_idx (block-major), col_idx and pair_pos (query-major).  One wavefront per 64 queries,
// lane = query; a ballot per block gives every query its rank inside the wavefront.
// Bound by the walk over the blocks (a ballot, a rank and two predicated stores each), so it is taken as seldom as the LDS allows:
// 16-bit entries in a window of 4096, 40 KB per workgroup, against block and place (6 bytes) in one of 2048, 48 KB.
// 12 heads x 112 320 tokens x 288 blocks: 785 -> 340 us; whole selection, 12 heads x
// 28 520 x 165: 498 -> 435 us, 32 760 x 84 (which one window held before): 247 -> 239 us.
// The walk is 9 vector instructions per block instead of 16 (a word's next bit is its sign, the ballot is the predicate, the block's start a
// scalar address, no position is tested when the run fits the window): 325 -> 267 us, 35 -> 29 at 32 760 x 84, 14 -> 11.7 at 32 x 6601 x 36.
// 0.94 GB of lists and masks take 180 of the 267.
__global__ __launch_bounds__(256) void fill_lists_kernel(const unsigned int* __restrict__ mask, int* __restrict__ row_ptr,
                                                         const int* __restrict__ wbase,
                                                         const int* __restrict__ blk_ptr, const int* __restrict__ wcnt,
                                                         int* __restrict__ q_idx, int* __restrict__ col_idx,
                                                         int* __restrict__ pair_pos, int S, int nb, int n_waves,
                                                         long long cap) {
    // The query-major entries of a wavefront's 64 rows form one contiguous run of col_idx / pair_pos.  They are collected
    // in LDS, a window of FILL_STAGE entries at a time, and written out as whole runs; a lane writing its own row's
    // entries straight to global memory touches a different cache line in every lane of every store.  A run longer
    // than the window walks the blocks once per window.  An entry is kept as block * 64 + rank among the wavefront's
    // queries in the block, 16 bits; its place in the block-major list is that rank plus the wavefront's start in the
    // block, looked up when the entry is written out.
    constexpr int FILL_STAGE = 4096;
    static_assert(VMOBA_MAX_BLOCKS * 64 <= 65536, "block and rank share 16 bits");
    __shared__ unsigned short sEnt[4][FILL_STAGE];
    __shared__ int sBase[4][VMOBA_MAX_BLOCKS];
    const int bh = blockIdx.y;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int w = xcd_contiguous(blockIdx.x, gridDim.x) * 4 + wv;
    if (w >= n_waves) return;                                            // no barrier below
    const int words = (nb + 31) / 32;
    // where this wavefront's entries of block j start in the block-major list: lane l keeps it for blocks l, l + 64, ...
    // (the walk below reads it with a lane broadcast: no LDS round trip inside the loop)
    int vbase[VMOBA_MAX_BLOCKS / 64];
#pragma unroll
    for (int i = 0; i < VMOBA_MAX_BLOCKS / 64; ++i) {
        const int j = lane + 64 * i;
        vbase[i] = 0;
        if (j < nb) sBase[wv][j] = vbase[i] = blk_ptr[(long long)bh * (nb + 1) + j] + wcnt[((long long)bh * nb + j) * n_waves + w];
    }
    const int q = w * 64 + lane;
    const bool live = q < S;
    unsigned int mw[VMOBA_MAX_MASK_WORDS];
#pragma unroll
    for (int wd = 0; wd < VMOBA_MAX_MASK_WORDS; ++wd)
        mw[wd] = (live && wd < words) ? mask[((long long)bh * S + q) * words + wd] : 0u;
    // row_ptr of the wavefront's rows: where the wavefront's run of the query-major lists starts (wbase, the scan of the
    // wavefronts' totals) plus the pairs of the lanes before; written here, row_ptr[S] by the offsets kernel
    int cnt = 0;
#pragma unroll
    for (int wd = 0; wd < VMOBA_MAX_MASK_WORDS; ++wd) cnt += __popc(mw[wd]);
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    const int run0 = wbase[(long long)bh * n_waves + w], n_run = __shfl(incl, 63, 64);   // the wavefront's run: [run0, run0 + n_run)
    if (live) row_ptr[(long long)bh * (S + 1) + q] = run0 + incl - cnt;
    // a head that kept more than `cap` pairs has an all-zero blk_ptr: no entry of its lists is ever read, and none is written
    if (row_ptr[(long long)bh * (S + 1) + S] > cap) return;
    int* const qi = q_idx + (long long)bh * cap;
    int* const ci = col_idx + (long long)bh * cap + run0;
    int* const pp = pair_pos + (long long)bh * cap + run0;
    // One walk over the blocks.  FIRST: it also writes the block-major list; ONLY: the run fits the window, so no position is tested.
    auto walk = [&](int win0, auto first, auto only) {
        constexpr bool FIRST = decltype(first)::value, ONLY = decltype(only)::value;
        int lr = incl - cnt - win0;                                      // position inside the window
        unsigned short* at = &sEnt[wv][0] + (ONLY ? lr : 0);
#pragma unroll
        for (int wd = 0; wd < VMOBA_MAX_MASK_WORDS; ++wd) {              // word by word, so that a word is one register
            if (wd * 32 >= nb) continue;
            unsigned int left = __brev(mw[wd]);                          // the next block's bit is the sign
            const int jn = __builtin_amdgcn_readfirstlane(min(32, nb - wd * 32));
            for (int b = 0; b < jn; ++b) {
                const unsigned long long bal = __ballot((int)left < 0);
                left += left;
                const unsigned rank = __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
                // the block's start is the same in every lane: a scalar address, and 32 bits of offset per lane
                int* const dst = FIRST ? qi + __builtin_amdgcn_readlane(vbase[wd >> 1], (wd & 1) * 32 + b) : nullptr;
                if (__builtin_amdgcn_inverse_ballot_w64(bal)) {
                    if (FIRST) dst[rank] = q;
                    const unsigned short entry = (unsigned short)((wd * 32 + b) * 64 + rank);
                    if (ONLY) {
                        *at++ = entry;
                    } else {
                        if ((unsigned)lr < (unsigned)FILL_STAGE) at[lr] = entry;
                        ++lr;
                    }
                }
            }
        }
    };
    for (int win0 = 0; win0 < n_run; win0 += FILL_STAGE) {
        if (n_run <= FILL_STAGE) walk(0, std::true_type{}, std::true_type{});
        else if (win0 == 0) walk(0, std::true_type{}, std::false_type{});
        else walk(win0, std::false_type{}, std::false_type{});
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        const int n = min(FILL_STAGE, n_run - win0);
        for (int i = lane; i < n; i += 64) {
            const int e = sEnt[wv][i];
            ci[win0 + i] = e >> 6;
            pp[win0 + i] = sBase[wv][e >> 6] + (e & 63);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

size_t score_long_lds_bytes(int D) { return (size_t)2 * 3 * LONG_KB * (D + 8) * 2 + ((size_t)HIST_BINS * 8 << LONG_COPIES); }

size_t score_lds_bytes(int nb, int D) {
    return (size_t)nb * D * 4 + (size_t)((QT * (nb | 1) + 1) & ~1) * 4 + HIST_BINS * 8 + 4 * QT * 4;
}

// What vmoba.h limits float32 calls by: score_lds_bytes with 12 KB of histogram, 3 KB more than the kernel takes.
size_t score_limit_bytes(int nb, int D) { return (size_t)nb * D * 4 + (size_t)QT * (nb | 1) * 4 + 12 * 1024; }

// The score kernels use more dynamic LDS than the default limit: raise a kernel's limit to the whole 160 KB of a
// compute unit, once per kernel (slot) and device.
int allow_full_lds(const void* kernel, int slot) {
    static std::mutex mu;
    static bool done[44][64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return VMOBA_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[slot][dev]) {
        if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return VMOBA_ERR_HIP;
        done[slot][dev] = true;
    }
    return VMOBA_OK;
}

int fix_shift_for(int64_t S) {
    int bits = 0;
    while (((int64_t)1 << bits) < S) ++bits;
    return 61 - bits;
}

}  // namespace

size_t vmoba_select_workspace_bytes(int B, int Hh, int64_t S, int nb) {
    return carve(nullptr, B * Hh, S, nb).total;
}

namespace {

// Host-side validation shared by the two entry points; everything that can be rejected without touching the device.
int select_args_ok(int B, int Hh, int64_t S, int D, int32_t n_blocks, const int32_t* blk_off, const vmoba_tensor* Qp,
                   const vmoba_tensor* Kp, float tau, float score_scale, int mode, int32_t topk, const float* Bmean,
                   const float* P, const uint32_t* mask, const int32_t* blk_ptr, const int32_t* q_idx,
                   const int32_t* row_ptr, const int32_t* col_idx, const int32_t* pair_pos, int64_t nnz_capacity,
                   const int64_t* k_out, const float* theta_out, const int32_t* dev_status) {
    if (B <= 0 || Hh <= 0 || S <= 0 || n_blocks <= 0 || nnz_capacity <= 0) return VMOBA_ERR_INVALID_ARG;
    if (!blk_off || !Bmean || !P || !mask || !blk_ptr || !q_idx || !row_ptr || !col_idx || !pair_pos ||
        !k_out || !theta_out || !dev_status)
        return VMOBA_ERR_INVALID_ARG;
    if (!tensor_ok(Qp) || !tensor_ok(Kp)) return VMOBA_ERR_INVALID_ARG;
    if (!std::isfinite(score_scale)) return VMOBA_ERR_INVALID_ARG;
    mode &= ~VMOBA_SELECT_OWN_BLOCK;
    if (mode < VMOBA_GLOBAL_THRESHOLD || mode > VMOBA_POOL_SOFTMAX_THRESHOLD) return VMOBA_ERR_UNSUPPORTED;
    const bool uses_tau = mode == VMOBA_GLOBAL_THRESHOLD || mode == VMOBA_LOCAL_THRESHOLD || mode == VMOBA_POOL_SOFTMAX_THRESHOLD;
    if (uses_tau && (!(tau > 0.f) || !(tau <= 1.f))) return VMOBA_ERR_INVALID_ARG;
    if (!uses_tau && topk < 1) return VMOBA_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return VMOBA_ERR_UNSUPPORTED;
    if (Qp->dtype != Kp->dtype) return VMOBA_ERR_UNSUPPORTED;
    if (n_blocks > VMOBA_MAX_BLOCKS || S > ((int64_t)1 << 30) || S * n_blocks > (int64_t)INT32_MAX)
        return VMOBA_ERR_UNSUPPORTED;
    return VMOBA_OK;
}

// The selection itself; `workspace` is the caller's buffer (vmoba_select) or the library's static one.
int select_impl(int B, int Hh, int64_t S, int D, int32_t n_blocks, const int32_t* blk_off,
                const vmoba_tensor* Qp, const vmoba_tensor* Kp, float tau, float score_scale,
                int mode, int32_t topk, float* Bmean, float* P, uint32_t* mask, int32_t* blk_ptr,
                int32_t* q_idx, int32_t* row_ptr, int32_t* col_idx, int32_t* pair_pos,
                int64_t nnz_capacity, int64_t* k_out, float* theta_out, int32_t* dev_status,
                const int32_t* query_pos, const int32_t* kv_rows, void* workspace, size_t workspace_bytes, void* stream) {
    {
        const int rc = select_args_ok(B, Hh, S, D, n_blocks, blk_off, Qp, Kp, tau, score_scale, mode, topk, Bmean, P, mask,
                                      blk_ptr, q_idx, row_ptr, col_idx, pair_pos, nnz_capacity, k_out, theta_out, dev_status);
        if (rc != VMOBA_OK) return rc;
    }
    if (!workspace) return VMOBA_ERR_INVALID_ARG;
    const bool own_block = (mode & VMOBA_SELECT_OWN_BLOCK) != 0;
    mode &= ~VMOBA_SELECT_OWN_BLOCK;
    const int* own_off = own_block ? blk_off : nullptr;
    const bool pool_softmax = mode == VMOBA_POOL_SOFTMAX_THRESHOLD;
    const bool bf16 = Qp->dtype == VMOBA_BF16;
    // LDS of the score kernel this call launches: bfloat16 queries go to the matrix-core kernel (block means as three
    // bfloat16 terms while they fit, as float32 up to 256 blocks, 64 blocks' terms at a time beyond), float32 queries to the plain FMA kernel
    const bool many = bf16 && n_blocks > 256;
    const int nb_pad = (n_blocks + 31) & ~31;
    // three bf16 terms of the means in LDS while they fit beside one copy of the histogram words and the accumulators fit
    // the registers (D = 128: up to 189 blocks; D = 64: 192), else the means as float32, split after every fetch
    const size_t lds_terms = (size_t)3 * (nb_pad > 128 ? n_blocks + 1 : nb_pad) * (D + 8) * 2;
    const bool fly = nb_pad > 192 || lds_terms + (size_t)HIST_BINS * 8 > 160 * 1024;
    const size_t lds_means = fly ? (size_t)nb_pad * (D + 4) * 4 : lds_terms;
    // the first radix level of the matrix-core kernel keeps up to 8 replicas of its 8 KB of histogram words, as many as fit
    int copy_shift = 3;
    while (copy_shift > 0 && lds_means + ((size_t)HIST_BINS * 8 << copy_shift) > 160 * 1024) --copy_shift;
    const size_t lds_mfma = lds_means + ((size_t)HIST_BINS * 8 << copy_shift);
    const size_t lds = many ? score_long_lds_bytes(D) : bf16 ? lds_mfma : score_lds_bytes(n_blocks, D);
    if ((bf16 ? lds : score_limit_bytes(n_blocks, D)) > 160 * 1024) return VMOBA_ERR_UNSUPPORTED;
    const int BH = B * Hh;
    SelectWs ws = carve(workspace, BH, S, n_blocks);
    if (workspace_bytes < ws.total) return VMOBA_ERR_WORKSPACE;
    if (ws.zero_bytes / 4 > (size_t)UINT32_MAX) return VMOBA_ERR_UNSUPPORTED;       // more than 10^5 heads in one call
    if (((uintptr_t)workspace) & 255) return VMOBA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const int n_waves = (int)ceil_div64(S, 64);
    const long long pool = (long long)S * n_blocks;
    // the pool sums to S (row soft-max) or to 1 (pool soft-max); the fixed-point scale leaves headroom for either
    const int fix_shift = pool_softmax ? fix_shift_for(2) : fix_shift_for(S);
    const double pool_total = pool_softmax ? 1.0 : (double)S;
    // target of the head-global cut: mass tau * S in fixed point (rounded up; tau >= 1 asks for more than the
    // pool can hold), or, for a fixed global k, the number of pairs topk * S
    unsigned long long target;
    if (mode == VMOBA_GLOBAL_TOPK) {
        target = (unsigned long long)std::min<long long>((long long)topk * S, pool);
    } else if (tau >= 1.f) {
        target = ~0ull;
    } else {
        target = (unsigned long long)std::ceil((double)tau * pool_total * (double)(1ull << fix_shift));
        if (target == 0) target = 1;
    }
    const TensorView Qv = make_view(Qp), Kv = make_view(Kp);

    // the block-mean kernel also clears the leading words of the workspace (histograms, head state)
#define LAUNCH_MEAN(BF, DD) block_mean_kernel<BF, DD><<<dim3(n_blocks, BH), dim3(256), 0, st>>>(Kv, blk_off, Bmean, Hh, n_blocks, kv_rows, (unsigned int*)workspace, (unsigned int)(ws.zero_bytes / 4))
    if (bf16 && D == 128) LAUNCH_MEAN(true, 128);
    else if (bf16 && D == 64) LAUNCH_MEAN(true, 64);
    else if (D == 128) LAUNCH_MEAN(false, 128);
    else LAUNCH_MEAN(false, 64);
#undef LAUNCH_MEAN
    VMOBA_CHECK_LAUNCH();

    float2* row_stat = pool_softmax ? ws.row_stat : nullptr;
    // pool soft-max: the radix levels run over the pool-normalised values, which only exist after the row statistics
    unsigned int* score_hist = pool_softmax ? nullptr : ws.hist_cnt;
    const int n_tiles = (int)ceil_div64(S, QT);
    // (float32 kernel) up to four tiles per workgroup, which loads the means once for them -- but not while compute units idle
    const int tiles_per_wg = (int)std::min<int64_t>(4, std::max<int64_t>(1, (int64_t)n_tiles * BH / (2 * vmoba_num_cus())));
    dim3 sgrid((unsigned)ceil_div64(n_tiles, tiles_per_wg), (unsigned)BH);
#define LAUNCH_SCORE(DD)                                                                                  \
    do {                                                                                                  \
        auto kfn = score_kernel<DD>;                                                                      \
        if (allow_full_lds((const void*)kfn, DD == 128 ? 0 : 1) != VMOBA_OK) return VMOBA_ERR_HIP;        \
        kfn<<<sgrid, dim3(256), lds, st>>>(Qv, Bmean, P, score_hist, ws.hist_sum, Hh, (int)S, n_blocks,   \
                                           score_scale, fix_shift, row_stat);                             \
    } while (0)
    if (bf16) {
        // one workgroup per compute unit (the LDS holds one), each with an equal share of all (head, query tile) pairs
        dim3 mgrid((unsigned)std::min<int64_t>((int64_t)BH * ceil_div64(S, SCORE_QT), vmoba_num_cus()));
#define LAUNCH_SCORE_MFMA_T(DD, FL, NM, TRV)                                                              \
    do {                                                                                                  \
        auto kfn = score_mfma_kernel<DD, FL, NM, TRV>;                                                    \
        if (allow_full_lds((const void*)kfn, 2 + (TRV ? 0 : 16) + (DD == 128 ? 0 : 8) + (FL ? 6 : NM - 1)) != VMOBA_OK) return VMOBA_ERR_HIP; \
        kfn<<<mgrid, dim3(SCORE_NT), lds, st>>>(Qv, Bmean, P, score_hist, ws.hist_sum, BH, Hh, (int)S, n_blocks, \
                                                score_scale, fix_shift, copy_shift, row_stat);            \
    } while (0)
        // rows of P that start 16-byte aligned take the kernel with the query on the lane, others the one with the block there
        // (not FLY: eight accumulator tiles leave no registers for the reduction's row values)
#define LAUNCH_SCORE_MFMA(DD, NM)                                                                         \
    do {                                                                                                  \
        if ((n_blocks & 3) == 0) LAUNCH_SCORE_MFMA_T(DD, false, NM, true);                                \
        else LAUNCH_SCORE_MFMA_T(DD, false, NM, false);                                                   \
    } while (0)
        // the bf16 terms fit: one instantiation per number of 32-block tiles
#define LAUNCH_SCORE_TILES(DD)                                                                            \
    do {                                                                                                  \
        switch ((n_blocks + 31) / 32) {                                                                   \
            case 1: LAUNCH_SCORE_MFMA(DD, 1); break;                                                      \
            case 2: LAUNCH_SCORE_MFMA(DD, 2); break;                                                      \
            case 3: LAUNCH_SCORE_MFMA(DD, 3); break;                                                      \
            case 4: LAUNCH_SCORE_MFMA(DD, 4); break;                                                      \
            case 5: LAUNCH_SCORE_MFMA(DD, 5); break;                                                      \
            default: LAUNCH_SCORE_MFMA(DD, 6); break;                                                     \
        }                                                                                                 \
    } while (0)
#define LAUNCH_SCORE_LONG_T(DD, NM, NW, SLOT)                                                             \
    do {                                                                                                  \
        auto kfn = score_long_kernel<DD, NM, NW>;                                                         \
        if (allow_full_lds((const void*)kfn, 34 + (DD == 128 ? 0 : 5) + SLOT) != VMOBA_OK) return VMOBA_ERR_HIP; \
        kfn<<<dim3((unsigned)std::min<int64_t>((int64_t)BH * ceil_div64(S, 32 * NW), vmoba_num_cus())), dim3(64 * NW), lds, st>>>( \
            Qv, Bmean, P, score_hist, ws.hist_sum, BH, Hh, (int)S, n_blocks, score_scale, fix_shift, row_stat); \
    } while (0)
        // more than 256 blocks: instantiations for 9, 10, 12, 14 and 16 tiles of 32 blocks
#define LAUNCH_SCORE_LONG(DD)                                                                             \
    do {                                                                                                  \
        if (n_blocks <= 288) LAUNCH_SCORE_LONG_T(DD, 9, 8, 0);                                            \
        else if (n_blocks <= 320) LAUNCH_SCORE_LONG_T(DD, 10, 4, 1);                                      \
        else if (n_blocks <= 384) LAUNCH_SCORE_LONG_T(DD, 12, 4, 2);                                      \
        else if (n_blocks <= 448) LAUNCH_SCORE_LONG_T(DD, 14, 4, 3);                                      \
        else LAUNCH_SCORE_LONG_T(DD, 16, 4, 4);                                                           \
    } while (0)
        if (many && D == 128) LAUNCH_SCORE_LONG(128);
        else if (many) LAUNCH_SCORE_LONG(64);
        else if (D == 128 && fly) LAUNCH_SCORE_MFMA_T(128, true, 0, true);
        else if (D == 128) LAUNCH_SCORE_TILES(128);
        else if (fly) LAUNCH_SCORE_MFMA_T(64, true, 0, true);
        else LAUNCH_SCORE_TILES(64);
#undef LAUNCH_SCORE_LONG
#undef LAUNCH_SCORE_LONG_T
#undef LAUNCH_SCORE_TILES
#undef LAUNCH_SCORE_MFMA
#undef LAUNCH_SCORE_MFMA_T
    } else if (D == 128) LAUNCH_SCORE(128);
    else LAUNCH_SCORE(64);
#undef LAUNCH_SCORE
    VMOBA_CHECK_LAUNCH();
    if (pool_softmax) {
        // the score kernel took no histogram in this mode: the first radix level is taken over G here
        pool_stat_kernel<<<dim3(BH), dim3(1024), 0, st>>>(ws.row_stat, ws.pool_stat, (int)S);
        VMOBA_CHECK_LAUNCH();
        pool_rescale_kernel<<<dim3((unsigned)std::min<int64_t>(ceil_div64(S, 4 * 8), 1024), (unsigned)BH), dim3(256), 0, st>>>(
            P, ws.row_stat, ws.pool_stat, ws.hist_cnt, ws.hist_sum, (int)S, n_blocks, fix_shift);
        VMOBA_CHECK_LAUNCH();
    }

    unsigned int* hc1 = ws.hist_cnt + (size_t)BH * HIST_BINS;
    unsigned int* hc2 = ws.hist_cnt + (size_t)2 * BH * HIST_BINS;
    unsigned long long* hs1 = ws.hist_sum + (size_t)BH * HIST_BINS;
    unsigned long long* hs2 = ws.hist_sum + (size_t)2 * BH * HIST_BINS;
    // at most 2^20 entries per workgroup (the packed histogram words), else as many workgroups as compute units
    const unsigned refine_gx = (unsigned)std::max<int64_t>(std::max<int64_t>(1, vmoba_num_cus() / BH), ceil_div64(pool, (int64_t)1 << 20));

    const unsigned wave_gx = (unsigned)ceil_div64(n_waves, 4);
    const bool local = mode == VMOBA_LOCAL_TOPK || mode == VMOBA_LOCAL_THRESHOLD;
    const int write_k = local ? 2 : (own_off ? 1 : 0);
    const bool small = !local && pool <= SMALL_POOL && S <= SMALL_ROWS && n_blocks <= SMALL_WORDS * 32;
    if (small) {
        auto kfn = mode == VMOBA_GLOBAL_TOPK ? small_cut_kernel<true> : small_cut_kernel<false>;
        kfn<<<dim3(BH), dim3(HIST_BINS), 0, st>>>(P, ws.hist_cnt, ws.hist_sum, target, fix_shift, mask, ws.wtot, ws.wcnt, blk_ptr, row_ptr,
                                                  (long long*)k_out, theta_out, dev_status, (int)S, n_blocks, n_waves, (long long)nnz_capacity,
                                                  own_off, query_pos, write_k);
        VMOBA_CHECK_LAUNCH();
    } else if (local) {
        const dim3 grid(wave_gx, BH);
        if (mode == VMOBA_LOCAL_TOPK) {
            // the fewest lanes per row that hold it with at most 64 columns each, in an instantiation per 8 columns
            int lpr_log2 = 0;
            while (n_blocks > 64 << lpr_log2) ++lpr_log2;
            const int cpl = ((n_blocks + (1 << lpr_log2) - 1) >> lpr_log2) + 7;
            decltype(&local_topk_kernel<8>) kfn[8] = {local_topk_kernel<8>, local_topk_kernel<16>, local_topk_kernel<24>, local_topk_kernel<32>,
                                                      local_topk_kernel<40>, local_topk_kernel<48>, local_topk_kernel<56>, local_topk_kernel<64>};
            kfn[cpl / 8 - 1]<<<grid, dim3(256), 0, st>>>(P, mask, ws.wtot, ws.wcnt, (int)S, n_blocks, n_waves, topk, lpr_log2, own_off, query_pos);
        } else {
            decltype(&local_threshold_kernel<1>) kfn[8] = {local_threshold_kernel<1>, local_threshold_kernel<2>, local_threshold_kernel<3>,
                                                           local_threshold_kernel<4>, local_threshold_kernel<5>, local_threshold_kernel<6>,
                                                           local_threshold_kernel<7>, local_threshold_kernel<8>};
            kfn[(n_blocks - 1) / 64]<<<grid, dim3(256), 0, st>>>(P, mask, ws.wtot, ws.wcnt, (int)S, n_blocks, n_waves, tau, own_off, query_pos);
        }
        VMOBA_CHECK_LAUNCH();
    } else {
#define SCAN_LEVEL(LV, HC, HS)                                                                                        \
    do {                                                                                                              \
        if (mode == VMOBA_GLOBAL_TOPK)                                                                                \
            scan_level_kernel<LV, true><<<dim3(BH), dim3(HIST_BINS), 0, st>>>(HC, HS, ws.state, target, fix_shift, pool, (long long*)k_out, theta_out, P, ws.ties, (int)S); \
        else                                                                                                          \
            scan_level_kernel<LV, false><<<dim3(BH), dim3(HIST_BINS), 0, st>>>(HC, HS, ws.state, target, fix_shift, pool, (long long*)k_out, theta_out, P, ws.ties, (int)S); \
    } while (0)
        SCAN_LEVEL(0, ws.hist_cnt, ws.hist_sum);
        VMOBA_CHECK_LAUNCH();
        refine_hist_kernel<1><<<dim3(refine_gx, BH), dim3(REFINE_NT), 0, st>>>(P, ws.state, hc1, hs1, pool, fix_shift, ws.ties, (int)S);
        VMOBA_CHECK_LAUNCH();
        SCAN_LEVEL(1, hc1, hs1);
        VMOBA_CHECK_LAUNCH();
        refine_hist_kernel<2><<<dim3(refine_gx, BH), dim3(REFINE_NT), 0, st>>>(P, ws.state, hc2, hs2, pool, fix_shift, ws.ties, (int)S);
        VMOBA_CHECK_LAUNCH();
        SCAN_LEVEL(2, hc2, hs2);
        VMOBA_CHECK_LAUNCH();
#undef SCAN_LEVEL
        // seldom anything to do (see last_kept_tie): no more workgroups than fill the chip, since 40 000 that return at once take 11 us.
        // With 0.14 million equal values a head, cut inside them, a whole selection of 12 heads x 32 760 tokens x 84 blocks takes 289 us (223 without
        // them), with 1.6 and 16 million 112 320 x 288 takes 3.74 and 5.10 ms (2.91); with up to 4096 workgroups a head all the same to 1 %.
        const unsigned row_gx = (unsigned)std::min<int64_t>(ceil_div64(S, 4 * 8), std::max(1, 8 * vmoba_num_cus() / BH));
        tie_count_kernel<<<dim3(row_gx, BH), dim3(256), 0, st>>>(P, ws.state, ws.ties, (int)S, n_blocks);
        VMOBA_CHECK_LAUNCH();
        row_scan_kernel<<<dim3(BH), dim3(SCAN_THREADS), 0, st>>>(ws.ties, ws.tie_base, ws.state, (int)S);
        VMOBA_CHECK_LAUNCH();
        mask_kernel<<<dim3(wave_gx, BH), dim3(256), 0, st>>>(P, ws.state, ws.tie_base, mask, ws.wtot, ws.wcnt,
                                                            (int)S, n_blocks, n_waves, own_off, query_pos);
        VMOBA_CHECK_LAUNCH();
    }
    if (!small && n_waves <= 64) {
        // rows of counts of at most 64 entries: one workgroup per head scans all of them, a launch less (69 -> 66 us with 49
        // wavefronts of queries and 40 blocks; with 200 and 80 it is 8 us slower)
        head_offsets_kernel<<<dim3(BH), dim3(1024), 0, st>>>(ws.wcnt, ws.wtot, blk_ptr, row_ptr, (long long*)k_out, theta_out, n_blocks, (int)S,
                                                             n_waves, (long long)nnz_capacity, dev_status, write_k);
        VMOBA_CHECK_LAUNCH();
    } else if (!small) {
        wave_scan_kernel<<<dim3(n_blocks + 1, BH), dim3(256), 0, st>>>(ws.wcnt, ws.wtot, ws.row_tot, n_blocks, n_waves);
        VMOBA_CHECK_LAUNCH();
        blk_ptr_kernel<<<dim3(BH), dim3(64), 0, st>>>(ws.row_tot, blk_ptr, row_ptr, (long long*)k_out, theta_out, n_blocks, (int)S,
                                                     (long long)nnz_capacity, dev_status, write_k);
        VMOBA_CHECK_LAUNCH();
    }
    fill_lists_kernel<<<dim3(wave_gx, BH), dim3(256), 0, st>>>(mask, row_ptr, ws.wtot, blk_ptr, ws.wcnt, q_idx, col_idx,
                                                              pair_pos, (int)S, n_blocks, n_waves,
                                                              (long long)nnz_capacity);
    VMOBA_CHECK_LAUNCH();
    return VMOBA_OK;
}

}  // namespace

extern "C" int vmoba_select(int B, int Hh, int64_t S, int D, int32_t n_blocks, const int32_t* blk_off,
                            const vmoba_tensor* Qp, const vmoba_tensor* Kp, float tau, float score_scale,
                            int mode, int32_t topk, float* Bmean, float* P, uint32_t* mask, int32_t* blk_ptr,
                            int32_t* q_idx, int32_t* row_ptr, int32_t* col_idx, int32_t* pair_pos,
                            int64_t nnz_capacity, int64_t* k_out, float* theta_out, int32_t* dev_status,
                            const int32_t* query_pos, const int32_t* kv_rows, void* workspace, size_t workspace_bytes, void* stream) {
    return select_impl(B, Hh, S, D, n_blocks, blk_off, Qp, Kp, tau, score_scale, mode, topk, Bmean, P, mask, blk_ptr, q_idx,
                       row_ptr, col_idx, pair_pos, nnz_capacity, k_out, theta_out, dev_status, query_pos, kv_rows, workspace,
                       workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------
// vmoba_select_static: vmoba_select for callers that cannot allocate.  Its scratch memory (histograms, head state,
// tie ranks, row and block counts) is a file-scope device array instead of a caller-provided workspace.  In host code
// the array's name is only a handle for the runtime: the device address is looked up once per device with
// hipGetSymbolAddress and that pointer is what the kernels get, exactly as they get the caller's workspace above.
static __device__ __align__(256) unsigned char scratch[VMOBA_SELECT_STATIC_MAX_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[MAX_DEVICES] = {};          // device address of `scratch` on each device, null until first use

int static_scratch_of_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return VMOBA_ERR_HIP;
    if (dev < 0 || dev >= MAX_DEVICES) return VMOBA_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return VMOBA_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return VMOBA_OK;
}

}  // namespace

extern "C" int vmoba_select_static(int B, int Hh, int64_t S, int D, int32_t n_blocks, const int32_t* blk_off,
                                   const vmoba_tensor* Qp, const vmoba_tensor* Kp, float tau, float score_scale,
                                   int mode, int32_t topk, float* Bmean, float* P, uint32_t* mask, int32_t* blk_ptr,
                                   int32_t* q_idx, int32_t* row_ptr, int32_t* col_idx, int32_t* pair_pos,
                                   int64_t nnz_capacity, int64_t* k_out, float* theta_out, int32_t* dev_status,
                                   const int32_t* query_pos, const int32_t* kv_rows, void* stream) {
    // everything that can be rejected on the host first, the size limit included
    const int rc = select_args_ok(B, Hh, S, D, n_blocks, blk_off, Qp, Kp, tau, score_scale, mode, topk, Bmean, P, mask,
                                  blk_ptr, q_idx, row_ptr, col_idx, pair_pos, nnz_capacity, k_out, theta_out, dev_status);
    if (rc != VMOBA_OK) return rc;
    if ((int64_t)B * Hh > (1 << 20)) return VMOBA_ERR_WORKSPACE;
    if (carve(nullptr, B * Hh, S, n_blocks).total > VMOBA_SELECT_STATIC_MAX_BYTES) return VMOBA_ERR_WORKSPACE;
    void* ws = nullptr;
    const int rs = static_scratch_of_current_device(&ws);
    if (rs != VMOBA_OK) return rs;
    return select_impl(B, Hh, S, D, n_blocks, blk_off, Qp, Kp, tau, score_scale, mode, topk, Bmean, P, mask, blk_ptr, q_idx,
                       row_ptr, col_idx, pair_pos, nnz_capacity, k_out, theta_out, dev_status, query_pos, kv_rows, ws,
                       VMOBA_SELECT_STATIC_MAX_BYTES, stream);
}
