// vmoba_attn_bwd: gradient of the block-sparse attention of Sec. 3.1 Step 3 with the selection
// held fixed.  With A the attention weights over the selected keys:
//   delta = rowsum(dO * O),  dV = A^T dO,  dP = dO V^T,  dS = A * (dP - delta),
//   dQ = scale * dS K,       dK = scale * dS^T Q.
//
// Three phases.  (1) delta (and what the other two need to know about their work).  (2) dQ: the forward's decomposition (tile of gathered
// queries x one key block), one partial dQ per (query, block) pair, summed query-major by a
// merge kernel.  (3) dK/dV: a workgroup owns a run of keys of one block and walks the whole
// query list of that block, so dK and dV of its keys stay in registers and are written once --
// no atomics anywhere, results are reproducible.  The attention weights are recomputed from
// Q, K and the forward's LSE in both (2) and (3).
#include "attn_common.h"
#include <type_traits>

#include <algorithm>
#include <cmath>

int64_t vmoba_max_tiles(int64_t cap, int TM);

namespace {

constexpr float LOG2E = 1.4426950408889634f;

// ---------------------------------------------------------------------------------------------
// What a backward call needs before its first large kernel, in one launch: workgroups with blockIdx.x below n_delta compute
// delta, the next ones write the flat tile list of the dQ kernel (256 tile ids each), the last one of every head the key
// runs of the dK/dV kernel.  (Four launches before; each of the small ones took about 5 us whatever its size.)
template <bool BF16, int D>
__device__ __forceinline__ void delta_rows(const TensorView& O, const TensorView& dO, const float* __restrict__ LSE, float* __restrict__ delta,
                                           const int* __restrict__ rows, char* __restrict__ dO_copy, int bh, int Hh, int S, int slot) {
    constexpr int EPP = BF16 ? 8 : 4;
    constexpr int LPQ = D / EPP;
    constexpr int QPW = 256 / LPQ;
    const int b = bh / Hh, h = bh % Hh;
    const int q = slot * QPW + threadIdx.x / LPQ;
    const int part = threadIdx.x % LPQ;
    float acc = 0.f;
    if (q < S) {
        // with a row map, O and dO are in the caller's token order and dO is also copied to block order
        const int qs = rows ? rows[q] : q;
        const char* po = O.ptr + ((long long)b * O.stride_b + (long long)qs * O.stride_s + (long long)h * O.stride_h) * (BF16 ? 2 : 4) + part * 16;
        const char* pd = dO.ptr + ((long long)b * dO.stride_b + (long long)qs * dO.stride_s + (long long)h * dO.stride_h) * (BF16 ? 2 : 4) + part * 16;
        const u32x4_t a = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(po));
        const u32x4_t c = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(pd));
        if (rows) *reinterpret_cast<u32x4_t*>(dO_copy + ((long long)bh * S + q) * D * (BF16 ? 2 : 4) + part * 16) = c;
        if constexpr (BF16) {
            acc = bf16lo_to_f32(a.x) * bf16lo_to_f32(c.x) + bf16hi_to_f32(a.x) * bf16hi_to_f32(c.x) +
                  bf16lo_to_f32(a.y) * bf16lo_to_f32(c.y) + bf16hi_to_f32(a.y) * bf16hi_to_f32(c.y) +
                  bf16lo_to_f32(a.z) * bf16lo_to_f32(c.z) + bf16hi_to_f32(a.z) * bf16hi_to_f32(c.z) +
                  bf16lo_to_f32(a.w) * bf16lo_to_f32(c.w) + bf16hi_to_f32(a.w) * bf16hi_to_f32(c.w);
        } else {
            acc = __uint_as_float(a.x) * __uint_as_float(c.x) + __uint_as_float(a.y) * __uint_as_float(c.y) +
                  __uint_as_float(a.z) * __uint_as_float(c.z) + __uint_as_float(a.w) * __uint_as_float(c.w);
        }
    }
#pragma unroll
    for (int off = LPQ / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (q < S && part == 0) {
        float* d = delta + (long long)bh * 2 * lse_delta_pitch(S) + q;
        d[0] = LSE[(long long)bh * S + q] * LOG2E;
        d[lse_delta_pitch(S)] = -acc;
    }
}

// Key-run table of one head.  A "run" is KPW consecutive keys of one block, the share of one dK/dV
// workgroup, and costs time in proportion to the length of the block's query list.  Workgroups are
// dispatched in index order, so the blocks are numbered longest list first (a longest-processing-time
// order: the short ones fill the tail of the launch): kb_order[r] = block at rank r,
// kb_start[r] = number of runs of the blocks at ranks 0..r-1.
// A last run of at most tail_max keys is not counted: the tail body takes those keys.
// slot_desc (bfloat16, instead of the other two): what the workgroup of a head's slot has to do, so that it learns it with one load and not
// with a search (it begins alone on its compute unit; search and look-ups took 7000 of the 30 000 cycles it spent outside its loop,
// beside 75 000 to 450 000 in it): {first key position, keys from there to the block's end, first list entry, list length}; slots past the
// runs are the blocks' tails, with TAIL_SLOT added to the number of keys; 0 keys: nothing.
constexpr int TAIL_SLOT = 1 << 30;
struct KeyRunLds { int cnt[VMOBA_MAX_BLOCKS]; int runs[VMOBA_MAX_BLOCKS]; int order[VMOBA_MAX_BLOCKS]; int start[VMOBA_MAX_BLOCKS]; int wave[4]; };
__device__ __forceinline__ void write_key_runs(KeyRunLds& lds, const int* __restrict__ blk_off, const int* __restrict__ blk_ptr,
                                               int* __restrict__ kb_start, int* __restrict__ kb_order, int4* __restrict__ slot_desc, int slots, int bh, int nb,
                                               int KPW, int tail_max) {
    const int t = threadIdx.x;
    const int* bp = blk_ptr + (long long)bh * (nb + 1);
    for (int j = t; j < nb; j += 256) lds.cnt[j] = bp[j + 1] - bp[j];
    __syncthreads();
    for (int j = t; j < nb; j += 256) {
        const int cnt = lds.cnt[j];
        int rank = 0;
        for (int i = 0; i < nb; ++i) rank += (lds.cnt[i] > cnt || (lds.cnt[i] == cnt && i < j)) ? 1 : 0;
        if (slot_desc) lds.order[rank] = j;
        else kb_order[(long long)bh * nb + rank] = j;
        const int L = blk_off[j + 1] - blk_off[j];
        const int tail = L % KPW;
        lds.runs[rank] = (tail > 0 && tail <= tail_max) ? L / KPW : (L + KPW - 1) / KPW;
    }
    __syncthreads();
    const int r0 = 2 * t < nb ? lds.runs[2 * t] : 0, r1 = 2 * t + 1 < nb ? lds.runs[2 * t + 1] : 0;
    int total;
    const int excl = block_exclusive_sum256(r0 + r1, lds.wave, &total);
    if (slot_desc) {
        if (2 * t < nb) lds.start[2 * t] = excl;
        if (2 * t + 1 < nb) lds.start[2 * t + 1] = excl + r0;
        __syncthreads();
        for (int i = t; i < slots; i += 256) {
            int4 d = make_int4(0, 0, 0, 0);
            int lo = i - total;                // rank of the slot's block
            if (i < total) {
                int hi = nb;                   // largest rank with start[rank] <= i
                lo = 0;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (lds.start[mid] <= i) lo = mid; else hi = mid;
                }
            }
            if (lo < nb) {
                const int j = lds.order[lo], L = blk_off[j + 1] - blk_off[j], tail = L % KPW;
                if (i < total) d = make_int4(blk_off[j] + (i - lds.start[lo]) * KPW, L - (i - lds.start[lo]) * KPW, bp[j], lds.cnt[j]);
                else if (tail <= tail_max) d = make_int4(blk_off[j] + L - tail, tail ? tail + TAIL_SLOT : 0, bp[j], lds.cnt[j]);
            }
            slot_desc[(long long)bh * slots + i] = d;
        }
        return;
    }
    int* out = kb_start + (long long)bh * (nb + 1);
    if (2 * t < nb) out[2 * t] = excl;
    if (2 * t + 1 < nb) out[2 * t + 1] = excl + r0;
    if (t == 0) out[nb] = total;
}

template <bool BF16, int D>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(TensorView O, TensorView dO, const float* __restrict__ LSE, float* __restrict__ delta, const int* __restrict__ rows,
                                                          char* __restrict__ dO_copy, const int* __restrict__ blk_ptr,
                                                          const int* __restrict__ blk_off, const int* __restrict__ head_tiles, int4* __restrict__ flat_desc, int* __restrict__ n_tiles,
                                                          int* __restrict__ clear, int* __restrict__ kb_start, int* __restrict__ kb_order, int4* __restrict__ slot_desc, int slots,
                                                          int BH, int Hh, int S, int nb, int TM, int KPW, int tail_max, int n_delta) {
    __shared__ union { TileListLds tiles; KeyRunLds runs; } lds;
    const int bh = blockIdx.y, x = blockIdx.x;
    if (x < n_delta) delta_rows<BF16, D>(O, dO, LSE, delta, rows, dO_copy, bh, Hh, S, x);
    else if (x + 1 < (int)gridDim.x) write_tile_list(lds.tiles, blk_ptr, blk_off, head_tiles, flat_desc, n_tiles, bh, BH, nb, TM, (x - n_delta) * 256);
    else {
        if (threadIdx.x < 2)
            delta[((long long)bh * 2 + threadIdx.x) * lse_delta_pitch(S) + S] = threadIdx.x == 0 ? INFINITY : 0.f;
        if (clear && bh == 0 && threadIdx.x == 2) *clear = 0;
        write_key_runs(lds.runs, blk_off, blk_ptr, kb_start, kb_order, BF16 ? slot_desc : nullptr, slots, bh, nb, KPW, tail_max);
    }
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA dQ tile kernel.  Same decomposition and operand orientation as the forward tile
// kernel (query = MFMA column); 4 wavefronts x 32 gathered queries, key chunks of 64:
//   S^T  = K . Q^T                    A = K rows (LDS),  B = Q^T (registers)
//   dP^T = V . dO^T                   A = V rows (LDS),  B = dO^T (registers)
//   dS^T = P^T * (dP^T - delta)       in registers, packed to bf16 as the next B operand
//   dQ^T += K^T . dS^T                A = K^T by transpose reads of the same K tile
//
// The key chunks pass through two LDS buffers, requested one chunk ahead straight from global memory (no registers hold rows in
// flight; one barrier per chunk); -delta is the value the sum for dP starts from, only a block's last chunk is masked.
// What bounds it: inside its loop, two workgroups per compute unit keep the matrix pipes busy for 90 % of the cycles, and the card's power limit
// holds the clock at 1.6-1.8 GHz meanwhile, so the products are on the 16-row instruction, which does the same work with less power
// (RowTile16; every operand feeds two of them, one per 16 queries).  A quarter of a workgroup's time lies before and behind the loop.
// Backward call, 480p, 12 heads, 1D / 2D / 3D partition: 4.13 / 4.18 / 3.23 -> 4.05 / 4.00 / 3.18 ms (dQ kernel -5 %); 2 x 6601 x 16 x 64: 520 -> 511 us
// (there as much by rows that lie free of bank conflicts).
template <int D>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_mfma_kernel(
    TensorView Q, TensorView K, TensorView V, TensorView dO, const float* __restrict__ lse_delta,
    const int* __restrict__ q_idx, const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles, float* __restrict__ dQpart, int Hh, int S,
    long long cap, float scale_log2, const int* __restrict__ kv_rows) {
    using TL = RowTile16<D>;
    constexpr int KC = 64;                      // keys per chunk
    constexpr int KSTEPS = D / 32, CT = D / 16;  // k-steps of the first two products, channel tiles of the third
    constexpr int HB = TL::HB, RB = TL::RB, PPR = TL::PPR, RPI = TL::RPI;
    constexpr int BUF = 4 * HB;                 // a chunk: 64 rows of K, then 64 rows of V
    constexpr int IPW = KC / RPI / 4;           // requests per wavefront, tensor and chunk
    __shared__ __align__(1024) char smem[2 * BUF];
    // The gathered rows of Q and dO pass through the second buffer on their way in; the wavefront's 32 partial rows, through the
    // first on their way out: written as the accumulators hold them, read back as whole rows.
    constexpr int OPITCH = D * 2 + 16;
    static_assert(4 * 32 * RB == BUF && 4 * 32 * OPITCH <= 2 * BUF, "rows of the four wavefronts fit a buffer, and both");

    Tile tc;
    if (!take_tile(flat_desc, n_tiles, tc)) return;
    const int bh = tc.bh, b = bh / Hh, h = bh % Hh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, l16 = lane & 15, g = lane >> 4;
    const long long seg = (long long)bh * cap;

    const int ent = wave * 32 + l32;
    const int e = min(ent, tc.count - 1);
    const int q = q_idx[seg + tc.list0 + e];
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    const char* kbase = K.ptr + ((long long)b * K.stride_b + (long long)h * K.stride_h) * 2;
    const char* vbase = V.ptr + ((long long)b * V.stride_b + (long long)h * V.stride_h) * 2;
    // row strides in bytes: below 2^24 and rows below 2^24, so a row's offset is one 24-bit multiply (host-checked)
    const uint32_t kss = (uint32_t)(K.stride_s * 2), vss = (uint32_t)(V.stride_s * 2);
    static_assert(IPW % TL::NPC == 0, "the same for every wavefront");
    uint32_t pc16[TL::NPC];
#pragma unroll
    for (int i = 0; i < TL::NPC; ++i) pc16[i] = TL::request_piece(lane, i);
    const int n_chunks = (tc.L + KC - 1) / KC;
    // Requests of a chunk: request i of this wavefront fetches rows (wave * IPW + i) * RPI + lane / PPR of it, of K and of V.
    // krow: where these keys lie -- the key positions themselves or, with keys in place, what kv_rows says, looked up one chunk
    // before the rows are requested.
    uint32_t krow[IPW];
    auto lookup_rows = [&](int c) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const uint32_t pos = (uint32_t)(tc.k0 + min(c * KC + (wave * IPW + i) * RPI + lane / PPR, tc.L - 1));
            krow[i] = kv_rows ? (uint32_t)kv_rows[pos] : pos;
        }
    };
    auto request = [&](int c, int i, int tensor) {
        const uint32_t l = lds0 + (uint32_t)(c & 1) * BUF + (uint32_t)(wave_u * IPW + i) * 1024;
        if (tensor == 0) dma_row16<0>(kbase, krow[i], kss, pc16[i % TL::NPC], l);
        else dma_row16<2 * HB>(vbase, krow[i], vss, pc16[i % TL::NPC], l);
    };
    // The wavefront's 32 gathered rows of Q, then those of dO, go to LDS as whole rows as well (one request covers 4 (8)
    // rows instead of a 32-byte piece of 32 rows); laid out like the key rows.  A wavefront reads back only what it requested: no barrier.
    const uint32_t g0 = lds0 + BUF + (uint32_t)wave_u * 32 * RB;
    auto gather = [&](const char* base, uint32_t stride) {
#pragma unroll
        for (int k = 0; k < 32 / RPI; ++k) {
            const int r = k * RPI + lane / PPR;
            const uint32_t pc = TL::request_piece(lane, k);
            dma16(base, __umul24((uint32_t)__shfl(q, r, 64), stride) + pc, g0 + k * 1024);
        }
    };
    auto fragments = [&](bf16x8_t (&f)[2][KSTEPS]) {       // queries l16 and 16 + l16
        const char* mine = smem + BUF + wave_u * 32 * RB + l16 * RB;
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks)
                f[qt][ks] = *reinterpret_cast<const bf16x8_t*>(mine + qt * 16 * RB + ((4 * ks + g) ^ TL::swz(l16)) * 16);
    };
    bf16x8_t qf[2][KSTEPS], dof[2][KSTEPS];
    lookup_rows(0);
    gather(Q.ptr + ((long long)b * Q.stride_b + (long long)h * Q.stride_h) * 2, (uint32_t)(Q.stride_s * 2));
    float lse2[2];
    f32x4_t ndl[2];                            // -delta, the value the sums for dP start from
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        const int qq = __shfl(q, qt * 16 + l16, 64);
        lse2[qt] = lse_delta[(long long)bh * 2 * lse_delta_pitch(S) + qq];
        const float d = lse_delta[((long long)bh * 2 + 1) * lse_delta_pitch(S) + qq];
        ndl[qt] = f32x4_t{d, d, d, d};
    }
    VMOBA_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    fragments(qf);
    __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0): the fragments have been read, their place is free
    asm volatile("" ::: "memory");
    gather(dO.ptr + ((long long)b * dO.stride_b + (long long)h * dO.stride_h) * 2, (uint32_t)(dO.stride_s * 2));
#pragma unroll
    for (int i = 0; i < IPW; ++i) { request(0, i, 0); request(0, i, 1); }
    lookup_rows(1);

    const f32x4_t zero4 = {0.f, 0.f, 0.f, 0.f};
    f32x4_t dqacc[CT][2];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) dqacc[ct][0] = dqacc[ct][1] = zero4;
    uint32_t rlane[TL::NRB], tlane[TL::NTB];
#pragma unroll
    for (int i = 0; i < TL::NRB; ++i) rlane[i] = TL::row_lane(lane, i);
#pragma unroll
    for (int i = 0; i < TL::NTB; ++i) tlane[i] = TL::tr_lane(lane, i);

    // A 32-key group is a sequence of units with one LDS operand and two matrix instructions (one per 16 queries) each: S^T over (16 keys,
    // k-step), dP^T over the same (with P = exp(S - LSE) computed between them, and dS of the first 16 keys), then the third product over the
    // channel tiles.  The operands pass through one ring of AHEAD + 1 registers, fetched AHEAD units before use, across the phases and into the
    // next group; fences keep that order, so no matrix instruction waits a full LDS round trip.
    constexpr int NP = 2 * KSTEPS;              // units of a phase
    static_assert(NP == CT, "as many units in each phase");
    constexpr int NSEQ = 3 * NP, VPU = 16 / NP; // VPU: values per unit of the middle phase
    constexpr int AHEAD = 3, RING = AHEAD + 1;
    static_assert(NSEQ % RING == 0, "the second group continues the ring where the first one left it");
    auto fetch = [&](uint32_t buf, int mt, int n) -> bf16x8_t {     // operand of unit n of group mt (n past the end: next group)
        if (n >= NSEQ) { mt += 1; n -= NSEQ; }
        if (n < NP) return TL::rows(smem, rlane, buf + mt * HB, n / KSTEPS, n % KSTEPS);
        if (n < 2 * NP) return TL::rows(smem, rlane, buf + (2 + mt) * HB, (n - NP) / KSTEPS, n % KSTEPS);
        return TL::transposed(smem, tlane, buf + mt * HB, n - 2 * NP);
    };
    VMOBA_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    fragments(dof);
    __syncthreads();                           // the first chunk has landed, the second buffer is free
    // MASK: the block ends inside the chunk (keys past the end get weight 0).  A separate body, because as a condition inside
    // one body it costs every 32-key group 45 predicated instructions beside its 24 matrix instructions.
    auto chunk = [&](int c, auto mask_tag) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_tag)::value;
        const uint32_t buf = (uint32_t)(c & 1) * BUF;
        const bool more = c + 1 < n_chunks;
        if (more) {
#pragma unroll
            for (int i = 0; i < IPW; ++i) { request(c + 1, i, 0); request(c + 1, i, 1); }
            lookup_rows(c + 2);
        }
        const int valid = tc.L - c * KC;
        bf16x8_t op[RING];
#pragma unroll
        for (int n = 0; n < RING; ++n) op[n] = fetch(buf, 0, n < AHEAD ? n : 0);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            if (!MASK || mt * 32 < valid) {
                f32x4_t s[2][2], dp[2][2];            // [16 keys][16 queries]: value i is key 16 * kt + 4 * g + i
                bf16x8_t dsf[2];
                const int vh = valid - mt * 32 - 4 * g;       // MASK: value (kt, i) belongs to a key of the block when 16 * kt + i < vh
                auto p_value = [&](int v) {           // S^T value -> P^T value, in place
                    const int kt = v >> 3, qt = (v >> 2) & 1, i = v & 3;
                    float p = exp2_raw(fmaf(s[kt][qt][i], scale_log2, -lse2[qt]));
                    if (MASK && 16 * kt + i >= vh) p = 0.f;
                    s[kt][qt][i] = p;
                };
                auto ds_value = [&](int v) {
                    const int kt = v >> 3, qt = (v >> 2) & 1, i = v & 3;
                    float d = s[kt][qt][i] * dp[kt][qt][i];
                    asm volatile("" : "+v"(d));
                    s[kt][qt][i] = d;
                };
#pragma unroll
                for (int n = 0; n < NSEQ; ++n) {
                    // the operand AHEAD units on (the group after the second one waits for the next chunk)
                    if (n + AHEAD < NSEQ || mt == 0) op[(n + AHEAD) % RING] = fetch(buf, mt, n + AHEAD);
                    const int m = n % NP, kt = m / KSTEPS, ks = m % KSTEPS;
                    if (n == 2 * NP) {
#pragma unroll
                        for (int v = 8; v < 16; ++v) ds_value(v);
#pragma unroll
                        for (int qt = 0; qt < 2; ++qt) {
                            const float d8[8] = {s[0][qt][0], s[0][qt][1], s[0][qt][2], s[0][qt][3], s[1][qt][0], s[1][qt][1], s[1][qt][2], s[1][qt][3]};
                            dsf[qt] = pack8(d8);
                        }
                    }
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt) {
                        if (n < NP)
                            s[kt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[n % RING], qf[qt][ks], ks == 0 ? zero4 : s[kt][qt], 0, 0, 0);
                        else if (n < 2 * NP)
                            dp[kt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[n % RING], dof[qt][ks], ks == 0 ? ndl[qt] : dp[kt][qt], 0, 0, 0);
                        else
                            dqacc[m][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[n % RING], dsf[qt], dqacc[m][qt], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (n >= NP && n < 2 * NP) {
#pragma unroll
                            for (int v = m * VPU + qt * VPU / 2; v < m * VPU + (qt + 1) * VPU / 2; ++v) {
                                p_value(v);
                                if (m >= NP / 2) ds_value(v - 8);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            }
        }
        VMOBA_WAIT_VMCNT(0);                   // the next chunk has landed (this wavefront's share)
        __syncthreads();
    };
    const int n_full = tc.L / KC;
    for (int c = 0; c < n_full; ++c) chunk(c, std::false_type{});
    if (n_full < n_chunks) chunk(n_full, std::true_type{});
    {
        // the tile's partials are consecutive rows of dQpart (bfloat16): stores of 1 KB runs instead of 16-byte pieces
        char* mine = smem + wave * 32 * OPITCH;                               // this wavefront's rows only: no barrier
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int qt = 0; qt < 2; ++qt) {
                u32x2_t v;
                v.x = pack_bf16x2(dqacc[ct][qt][0], dqacc[ct][qt][1]);
                v.y = pack_bf16x2(dqacc[ct][qt][2], dqacc[ct][qt][3]);
                *reinterpret_cast<u32x2_t*>(mine + (qt * 16 + l16) * OPITCH + (ct * 16 + g * 4) * 2) = v;
            }
        char* dst = reinterpret_cast<char*>(dQpart) + (seg + tc.list0) * (long long)(D * 2);
        constexpr int LPR = D * 2 / 16;                                       // lanes per row
#pragma unroll
        for (int k = 0; k < 32 * LPR / 64; ++k) {
            const int row = k * (64 / LPR) + lane / LPR, piece = lane % LPR;
            const u32x4_t x = *reinterpret_cast<const u32x4_t*>(mine + row * OPITCH + piece * 16);
            const int e2 = wave * 32 + row;
            if (e2 < tc.count) *reinterpret_cast<u32x4_t*>(dst + (long long)e2 * (D * 2) + piece * 16) = x;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA dK/dV kernel.  A workgroup owns 128 consecutive keys of one block (key = MFMA column = lane % 32) and walks
// the block's query list in half-chunks of 32 gathered queries.
//   S   = Q . K^T      A = Q rows (LDS),   B = K^T (registers, loaded once)
//   dP  = dO . V^T     A = dO rows (LDS),  B = V^T (registers, loaded once)
//   dV^T += dO^T . P   A = dO^T by transpose reads of the dO tile,  B = P packed from S
//   dK^T += Q^T . dS   A = Q^T  by transpose reads of the Q tile,   B = dS
// What limits such a kernel is the LDS issue rate (one operand fetch per matrix instruction, two
// for a transposed operand), not the matrix pipe.  So the 128 keys are held by two PAIRS of
// wavefronts with 64 keys (two 32-key groups) each, and the two wavefronts of a pair split the products:
//   wavefront 0 of the pair:  S  = Q  . K^T  ->  P = exp(S - LSE)  ->  dV^T += dO^T . P
//   wavefront 1 of the pair:  dP - delta = dO . V^T - delta  ->  dS = P * (dP - delta)  ->  dK^T += Q^T . dS
// so every operand fetched from LDS feeds two matrix instructions (one per key group), and each
// wavefront keeps only one set of fragments (K or V) and one accumulator tile (dV^T or dK^T).
// P travels from wavefront 0 to wavefront 1 as packed bf16 through a small LDS buffer (same lane,
// same accumulator layout on both sides); wavefront 1 therefore runs the same pipeline one
// half-chunk later, and the steps are separated by one workgroup barrier per half-chunk.
// Step hc of the workgroup, local step t = hc - (wavefront % 2), all interleaved:
//   matrix:  S or dP of half-chunk t + 1,  dV or dK of half-chunk t - 1      vector: P or dS of t
//   memory:  rows, LSE and delta of half-chunk hc + 5, list entries of half-chunk hc + 8, straight into LDS.
// The rows are requested by wavefronts 1 alone: wavefronts 0 have the exponentials and were 200 of 1740 cycles behind at every barrier
// (now 1650 cycles a step, 1024 of them matrix instructions; the clock is at 1.57 GHz then, 2.4 without load).  -delta is the value the sums for dP
// start from: 32 additions a step less (by itself 0.3 % of a training step).  Backward calls of 14 040 tokens x 12 heads x 128 / 2 x 6601 x 16 x 64, with the slot descriptors
// and the row-wise output: 737 / 540 -> 720 / 521 us; 480p, 1D / 2D / 3D: -1 / -1 / -2 %.
//
// Everything the walk reads goes from global memory to LDS without passing through registers (global_load_lds): rings of
// eight half-chunks of Q and dO rows, of their LSE and delta (accumulator order) and of the list entries, from which a lane
// takes the row number it requests.  A half-chunk h is read from the end of step h - 2 to step h + 2 and its slot is
// requested again in step h + 3; a step ends with a wait for what was requested up to two steps before, then the barrier,
// so what step s requested is visible from step s + 3 on.  The loop holds no other global loads, so the count of
// the wait is exact.  (Before: staged through registers -- 8 row loads and 8 LDS writes per wavefront and chunk of
// 64, 32 registers of rows in flight and the copies from and to the accumulator registers that these forced, 7.1 and 8.6
// instructions per matrix instruction for the two wavefronts of a pair, 6.0 and 7.7 then and, with the above, 5.5 and 5.9 now.  480p, 12 heads, 1D / 2D / 3D partition:
// 2.80 / 2.66 / 2.13 -> 2.62 / 2.46 / 2.00 ms.  Timing variants of this form: without the row requests -5 %, without the
// barrier as well -11 %, without the operand reads from LDS -13 %: no single limiter.)
// Rows past the end of the list repeat its last entry; their LSE is +inf (weight 0) and their delta 0, read from a
// spare element behind the head's S values.
//
// A wavefront issues in order and a matrix instruction occupies the matrix pipe for 32 cycles, so the step is cut
// into units of one matrix instruction followed by an equal share of the vector, LDS and memory instructions,
// with scheduling fences between them (two matrix instructions back to back would stall the second one while
// the vector unit idles).  Operands are fetched two k-steps (eight units) before use.  The first LEAD units of a
// step carry no vector work: it needs P and LSE / delta, which are only requested from LDS at the start of the step.
// S / dP of even and odd half-chunks live in two register sets that swap roles, so no accumulator is ever copied.
template <int D>
struct DkvLds : RowTile<D> {
    using RowTile<D>::HB;
    static constexpr int NS = 8;                                       // half-chunks per ring
    static constexpr int LD0 = 2 * NS * HB;                            // LSE and delta: [NS][64] floats
    static constexpr int IX0 = LD0 + NS * 64 * 4;                      // list entries: [NS + 1][32]; a request fills two half-chunks
    static constexpr int X0 = IX0 + (NS + 1) * 32 * 4;                 // packed P: [pair][step parity][key group * 2 + s][lane]
    static constexpr int BYTES = X0 + 2 * 2 * 4 * 64 * 16;
    static_assert(X0 % 16 == 0 && BYTES <= 160 * 1024, "LDS of one compute unit");
};

// Matrix instruction on a sum that stays in accumulator registers.  (This file is compiled so that the results of the matrix
// instructions it does not name in assembly go to ordinary registers: S and dP are read by vector instructions, which cannot
// read accumulator registers -- with the compiler's choice for a kernel of this size, everything there, every one of
// their values takes a copy, one instruction more per matrix instruction.)  The compiler sees neither that such an instruction needs
// two wait states after a vector instruction that wrote one of its operands, nor how long its result takes: a pack that
// feeds one lies whole units before it, and acc_ready stands between the last of them and everything else that touches the sums.
// (tests/test_matrix_wait_states.py follows the compiled code for both.)
__device__ __forceinline__ void mfma_acc(f32x16_t& d, bf16x8_t a, bf16x8_t b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void acc_ready(f32x16_t (&d)[2][2]) {
    asm volatile("s_nop 15" : "+a"(d[0][0]), "+a"(d[0][1]), "+a"(d[1][0]), "+a"(d[1][1]));
}
__device__ __forceinline__ void acc_ready(f32x16_t (&d)[2][4]) {
    asm volatile("s_nop 15" : "+a"(d[0][0]), "+a"(d[0][1]), "+a"(d[0][2]), "+a"(d[0][3]), "+a"(d[1][0]), "+a"(d[1][1]), "+a"(d[1][2]), "+a"(d[1][3]));
}

template <int D>
__device__ __forceinline__ void dkv_pair_body(
    char* smem, int bh, const int4 desc, const TensorView& Q, const TensorView& K, const TensorView& V, const TensorView& dO,
    const float* __restrict__ lse_delta, const int* __restrict__ q_idx, const TensorView& dK, const TensorView& dV, const int* __restrict__ rows,
    const int* __restrict__ kv_rows, int Hh, int S, long long cap, float scale_log2, float scale) {
    using TL = DkvLds<D>;
    constexpr int KSTEPS = D / 16, DT = D / 32, NST = KSTEPS;
    constexpr int IPW = 32 / TL::RPI / 2;     // row requests per wavefront 1 of a pair, tensor and half-chunk
    constexpr int NS = TL::NS, HB = TL::HB, GP = TL::GP;
    constexpr int NU = 4 * NST, LEAD = 4;     // units per step; units without vector work
    static_assert(NST == 2 * DT && NST % 4 == 0, "one k-step and one (s, dt) step per step, operand ring of four");

    // value v belongs to unit LEAD + v * (NU - LEAD) / 32: first value of unit n
    constexpr auto first_value = [](int n) { return n <= LEAD ? 0 : ((n - LEAD) * 32 + NU - LEAD - 1) / (NU - LEAD); };

    const int b = bh / Hh, h = bh % Hh;
    const int k0 = desc.x, L = desc.y;                  // first key position of the run, keys from there to the block's end
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pair = wave >> 1, role = wave & 1;
    const int l32 = lane & 31, hf = lane >> 5;
    const int kbase = pair * 64;                        // first key of the pair inside the run
    const bool pair_live = kbase < L;
    const int cnt = desc.w;
    const int* const list = q_idx + (long long)bh * cap + desc.z;
    const int first_entry = cnt > 0 ? list[min(tid, cnt - 1)] : 0;       // requested before the fragments: the rows wait for it

    // fragments of the pair's keys: K rows for wavefront 0, V rows for wavefront 1 (B operands, key = lane % 32)
    bf16x8_t frag[2][KSTEPS];
    {
        const TensorView& src = role == 0 ? K : V;
#pragma unroll
        for (int kg = 0; kg < 2; ++kg) {
            const int krow = k0 + min(kbase + kg * 32 + l32, L - 1);
            const long long kin = kv_rows ? kv_rows[krow] : krow;     // row of K / V that holds this key
            const char* sp = src.ptr + ((long long)b * src.stride_b + kin * src.stride_s + (long long)h * src.stride_h) * 2;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) frag[kg][ks] = *reinterpret_cast<const bf16x8_t*>(sp + (ks * 16 + hf * 8) * 2);
        }
    }
    f32x16_t acc[2][DT];                       // dV^T (wavefront 0) or dK^T (wavefront 1), [key group][channel tile]
#pragma unroll
    for (int kg = 0; kg < 2; ++kg)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[kg][dt][i] = 0.f;

    if (cnt > 0) {
        const char* qbase = Q.ptr + ((long long)b * Q.stride_b + (long long)h * Q.stride_h) * 2;
        const char* dobase = dO.ptr + ((long long)b * dO.stride_b + (long long)h * dO.stride_h) * 2;
        // row strides in bytes: below 2^24 and rows below 2^24, so a row's offset is one 24-bit multiply (host-checked)
        const uint32_t qss = (uint32_t)(Q.stride_s * 2), doss = (uint32_t)(dO.stride_s * 2);
        const uint32_t SP = (uint32_t)lse_delta_pitch(S);
        const char* ld_base = reinterpret_cast<const char*>(lse_delta + (long long)bh * 2 * SP);
        const int H = (cnt + 63) / 64 * 2;                  // half-chunks, an even number (see the register sets below)

        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
        const int* sIdx = reinterpret_cast<const int*>(smem + TL::IX0);
        const uint32_t pc16 = TL::request_piece(lane);
        const int idx_row = pair * IPW * TL::RPI + lane / TL::PPR;           // + i * RPI: row of request i this lane takes part in
        // LSE / delta: lanes 0..31 request LSE, lanes 32..63 delta; lane l % 32 = position p holds row ld_row (accumulator
        // order: the 16 values a lane half needs are contiguous)
        const int ld_row = ((l32 & 3) << 2) | (((l32 >> 2) & 1) << 1) | (((l32 >> 3) & 1) << 4) | (l32 >> 4);
        const uint32_t ld_hf = hf ? SP * 4 : 0;
        // requests of half-chunk x, piece by piece: row numbers from LDS, then LSE / delta, Q rows, dO rows
        uint32_t qn[IPW];
        uint32_t lq = 0;
        auto read_idx = [&](int x) {
            const int* p = sIdx + (x & (NS - 1)) * 32;
#pragma unroll
            for (int i = 0; i < IPW; ++i) qn[i] = (uint32_t)p[idx_row + i * TL::RPI];
        };
        auto read_ld_idx = [&](int x) { lq = (uint32_t)sIdx[(x & (NS - 1)) * 32 + ld_row]; };
        auto ld_offset = [&](int x) { return (32 * x + ld_row < cnt ? lq : (uint32_t)S) * 4 + ld_hf; };
        auto ld_slot = [&](int x) { return lds0 + TL::LD0 + (uint32_t)(x & (NS - 1)) * 256; };
        // Wavefront 0 of the first pair requests LSE / delta of half-chunk hc + 5, wavefront 0 of the second pair the list
        // entries of half-chunk hc + 8 (and, with what it will be filled with next, hc + 9) -- without a branch
        const bool lists = pair == 1;
        const char* const side_base = lists ? reinterpret_cast<const char*>(list) : ld_base;
        auto dma_side = [&](int hc) {
            const uint32_t e = (uint32_t)min(32 * (hc + 8) + lane, cnt - 1) * 4, l = ld_offset(hc + 5);
            dma4(side_base, lists ? e : l, lists ? lds0 + TL::IX0 + (uint32_t)(hc & (NS - 1)) * 128 : ld_slot(hc + 5));
        };
        const uint32_t lds_rows = lds0 + (uint32_t)pair * IPW * GP;
        auto dma_rows = [&](uint32_t off, int i, int tensor) {
            const uint32_t l = lds_rows + off + (uint32_t)i * GP;
            if (tensor == 0) dma_row16<0>(qbase, qn[i], qss, pc16, l);
            else dma_row16<NS * HB>(dobase, qn[i], doss, pc16, l);
        };
        auto request_all = [&](int hc) {
            if (role == 0) {
                read_ld_idx(hc + 5);
                dma_side(hc);
            } else {
                read_idx(hc + 5);
#pragma unroll
                for (int i = 0; i < IPW; ++i) { dma_rows((uint32_t)((hc + 5) & (NS - 1)) * HB, i, 0); dma_rows((uint32_t)((hc + 5) & (NS - 1)) * HB, i, 1); }
            }
        };
        // Ends a step: what this wavefront requested up to two steps before has landed, then everybody's.  A step makes
        // 2 * IPW requests (role 0: one more, first in the step).
        auto end_step = [&](auto role_tag) {
            VMOBA_WAIT_VMCNT(decltype(role_tag)::value == 0 ? 2 : 4 * IPW);
            __syncthreads();
        };
        // prologue: list entries of half-chunks 0..7, then rows of half-chunks 0..4, of which 0..2 have to be here
        reinterpret_cast<int*>(smem + TL::IX0)[tid] = first_entry;
        __syncthreads();
        read_ld_idx(wave);
        dma4(ld_base, ld_offset(wave), ld_slot(wave));
        if (wave == 0) { read_ld_idx(4); dma4(ld_base, ld_offset(4), ld_slot(4)); }
        if (role == 1) {
#pragma unroll
            for (int x = 0; x < 5; ++x) {
                read_idx(x);
#pragma unroll
                for (int i = 0; i < IPW; ++i) { dma_rows((uint32_t)x * HB, i, 0); dma_rows((uint32_t)x * HB, i, 1); }
            }
            VMOBA_WAIT_VMCNT(4 * IPW);
        } else {
            VMOBA_WAIT_VMCNT(0);
        }
        __syncthreads();

        const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // row operands come from the Q tile for wavefront 0 (S) and from the dO tile for wavefront 1 (dP);
        // transposed operands from the dO tile for wavefront 0 (dV) and from the Q tile for wavefront 1 (dK)
        uint32_t rlane[TL::NRB], tlane[2][TL::NTB];
#pragma unroll
        for (int k = 0; k < TL::NRB; ++k) rlane[k] = (role == 0 ? 0u : (uint32_t)(NS * HB)) + TL::row_lane(lane, k);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int dt = 0; dt < TL::NTB; ++dt) tlane[t][dt] = (role == 0 ? (uint32_t)(NS * HB) : 0u) + TL::tr_lane(lane, t, dt);
        auto half_off = [&](int half) { return (uint32_t)(half & (NS - 1)) * HB; };
        auto next_off = [&](uint32_t off) { return off == (NS - 1) * HB ? 0u : off + HB; };
        auto read_rows = [&](uint32_t off, int ks) { return TL::rows(smem, rlane, off, ks); };
        auto read_tr = [&](uint32_t off, int step) { return TL::transposed(smem, tlane, off, step / DT, step % DT); };

        if (pair_live) {
            f32x16_t xa[2] = {zero16, zero16}, xb[2] = {zero16, zero16};    // S or dP of the even / odd local half-chunks
            bf16x8_t w_prev[2][2];                          // packed P or dS of local half-chunk t - 1, [kg][s]
            {
                const f32x4_t z4 = {0.f, 0.f, 0.f, 0.f};
                const bf16x4_t zb = __builtin_convertvector(z4, bf16x4_t);
                const bf16x8_t z8 = __builtin_shufflevector(zb, zb, 0, 1, 2, 3, 4, 5, 6, 7);
                w_prev[0][0] = w_prev[0][1] = w_prev[1][0] = w_prev[1][1] = z8;
            }
            // LSE (wavefront 0) or -delta (wavefront 1) of a half-chunk's 32 rows, as the accumulators want them: the 16 of this lane half
            auto read_ld = [&](int half) {
                const f32x4_t* lp = reinterpret_cast<const f32x4_t*>(smem + TL::LD0 + (half & (NS - 1)) * 256 + role * 128 + hf * 64);
                f32x16_t r;
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const f32x4_t a4 = lp[g4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) r[g4 * 4 + u] = a4[u];
                }
                return r;
            };
            // S / dP of half-chunk 0; the sums for dP - delta start at -delta
            f32x16_t start = role == 0 ? zero16 : read_ld(0);
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                const bf16x8_t a = read_rows(0u, ks);
#pragma unroll
                for (int kg = 0; kg < 2; ++kg)
                    xa[kg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, frag[kg][ks], ks == 0 ? start : xa[kg], 0, 0, 0);
            }
            if (role == 1) start = read_ld(1);
            bf16x8_t rop[4], top[4];                        // operands of k-steps st .. st + 2, slot = k-step % 4
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                rop[k] = read_rows(HB, k);
                top[k] = read_tr(0u, k);                    // local step 0 multiplies them by zeros
            }
            // ring offsets of half-chunks t - 1 (step 0: 0, times zeros), t, t + 1, t + 2 and of the one whose rows are requested
            uint32_t o_prev = 0, o_cur = 0, o_1 = HB, o_2 = 2 * HB, o_req = half_off(5 + role);
            u32x4_t* xbuf = reinterpret_cast<u32x4_t*>(smem + TL::X0) + pair * 2 * 4 * 64 + lane;     // + parity * 256 + slot * 64

            // one local step; ROLE is compile-time
            // (x_cur holds S or dP of half-chunk t, x_nxt receives that of t + 1: the two sets swap roles every step)
            auto local_step = [&](int t, auto role_tag, f32x16_t(&x_cur)[2], f32x16_t(&x_nxt)[2]) {
                constexpr int ROLE = decltype(role_tag)::value;
                const int hc = t + ROLE;
                asm volatile("" : "+v"(x_cur[0]), "+v"(x_cur[1]));      // whole registers across the loop, not 32 values
                // wavefront 0: LSE of half-chunk t; wavefront 1: what the sums for dP of half-chunk t + 1 start from, read a step before
                const f32x16_t ld = ROLE == 0 ? read_ld(t) : start;
                u32x4_t pin[4];
                if constexpr (ROLE == 1) {
#pragma unroll
                    for (int sl = 0; sl < 4; ++sl) pin[sl] = xbuf[(t & 1) * 256 + sl * 64];
                }
                float w[2][16];
                float l[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) l[i] = ld[i];
                static_for<NU>([&](auto unit) __attribute__((always_inline)) {
                    constexpr int n = decltype(unit)::value, st = n >> 2, q = n & 3, kg = q >> 1;
                    constexpr int s2 = st + 2;                  // the k-step whose operands are fetched now
                    if (q == 0) rop[s2 & 3] = s2 < NST ? read_rows(o_1, s2) : read_rows(o_2, s2 - NST);
                    if (q == 1) top[s2 & 3] = s2 < NST ? read_tr(o_prev, s2) : read_tr(o_cur, s2 - NST);
                    if constexpr ((q & 1) == 0)
                        x_nxt[kg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rop[st & 3], frag[kg][st], st > 0 ? x_nxt[kg] : ROLE == 0 ? zero16 : ld, 0, 0, 0);
                    else
                        mfma_acc(acc[kg][st % DT], top[st & 3], w_prev[kg][st / DT]);
                    __builtin_amdgcn_sched_barrier(0);          // the matrix instruction leads its unit
                    // the unit's share of the 32 values of P or dS, in the order (s, channel of s, key group)
                    // (an ld passes through an empty assembly statement just before its turn: keeps the arithmetic on it in its unit)
                    constexpr int V0 = first_value(n), V1 = first_value(n + 1);
                    if constexpr (ROLE == 0 && n == LEAD - 1) asm volatile("" : "+v"(l[0]));
                    static_for<V1 - V0>([&](auto value) __attribute__((always_inline)) {
                        constexpr int v = V0 + decltype(value)::value, g2 = v & 1, i = v >> 1;
                        if constexpr (ROLE == 0) {
                            w[g2][i] = exp2_raw(fmaf(x_cur[g2][i], scale_log2, -l[i]));
                        } else {
                            const u32x4_t pk = pin[g2 * 2 + i / 8];
                            const uint32_t word = (i % 8) / 2 == 0 ? pk.x : (i % 8) / 2 == 1 ? pk.y : (i % 8) / 2 == 2 ? pk.z : pk.w;
                            const float pval = (i & 1) ? bf16hi_to_f32(word) : bf16lo_to_f32(word);
                            w[g2][i] = pval * x_cur[g2][i];
                        }
                        asm volatile("" : "+v"(w[g2][i]));
                        if constexpr (ROLE == 0 && g2 == 1 && i < 15) asm volatile("" : "+v"(l[i + 1]));
                    });
                    // packed operands are replaced when their values are complete and their last reader of this step has issued
                    constexpr int PACK0 = LEAD + 15 * (NU - LEAD) / 32;             // the unit of value 15
                    static_assert(PACK0 >= NU / 2 - 1, "the readers of the first half have issued");
                    if (n == PACK0 || n == NU - 1) {
                        const int sidx = n == NU - 1 ? 1 : 0;
#pragma unroll
                        for (int k2 = 0; k2 < 2; ++k2) {
                            w_prev[k2][sidx] = pack8(&w[k2][8 * sidx]);
                            if constexpr (ROLE == 0) {
                                u32x4_t o;
                                __builtin_memcpy(&o, &w_prev[k2][sidx], 16);
                                xbuf[(t & 1) * 256 + (k2 * 2 + sidx) * 64] = o;
                            }
                        }
                    }
                    if (ROLE == 1 && n == NU - 6) start = read_ld(t + 2);
                    // the step's requests
                    if (n == 1) {
                        if (ROLE == 0) read_ld_idx(hc + 5);
                        else read_idx(hc + 5);
                    }
                    if (ROLE == 0 && n == 5) dma_side(hc);
                    if (ROLE == 1 && (n & 1) == 0 && n >= 6 && n < 6 + 4 * IPW) dma_rows(o_req, (n - 6) / 4, ((n - 6) >> 1) & 1);
                    __builtin_amdgcn_sched_barrier(0);
                });
                o_prev = o_cur;
                o_cur = o_1;
                o_1 = o_2;
                o_2 = next_off(o_2);
                if (ROLE == 1) o_req = next_off(o_req);
            };
            using R0 = std::integral_constant<int, 0>;
            using R1 = std::integral_constant<int, 1>;
            // dV or dK of the last half-chunk, whose packed operand the last step left; nothing of S / dP outlives the loop.  These matrix
            // instructions are the compiler's: what it moves here it may move, and waits for.
            auto drain = [&]() {
                acc_ready(acc);
#pragma unroll
                for (int st = 0; st < NST; ++st) {
                    if (st + 2 < NST) top[(st + 2) & 3] = read_tr(o_prev, st + 2);
#pragma unroll
                    for (int kg = 0; kg < 2; ++kg)
                        acc[kg][st % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(top[st & 3], w_prev[kg][st / DT], acc[kg][st % DT], 0, 0, 0);
                }
            };
            if (role == 0) {
                for (int t = 0; t < H; t += 2) {
                    local_step(t, R0{}, xa, xb);
                    end_step(R0{});
                    local_step(t + 1, R0{}, xb, xa);
                    end_step(R0{});
                }
                drain();
            } else {
                request_all(0);
                for (int t = 0; t < H; t += 2) {
                    end_step(R1{});
                    local_step(t, R1{}, xa, xb);
                    end_step(R1{});
                    local_step(t + 1, R1{}, xb, xa);
                }
                drain();
            }
        } else {
            // a pair whose keys lie past the end of the block only helps to move rows
            for (int hc = 0; hc < H; ++hc) {
                request_all(hc);
                if (role == 0) end_step(std::integral_constant<int, 0>{});
                else end_step(std::integral_constant<int, 1>{});
            }
        }
        VMOBA_WAIT_VMCNT(0);                   // no request may reach LDS that belongs to another workgroup by then
    }
    // The sums leave through LDS (the rings are free): written as the accumulators hold them, 8 bytes per lane, read back as whole rows, so that
    // a store request is four (eight) whole rows instead of 16-byte pieces of 32.
    __syncthreads();
    if (pair_live) {
        constexpr int OPITCH = D * 2 + 16, LPR = D * 2 / 16;          // LPR: lanes per row
        static_assert(4 * 64 * OPITCH <= TL::BYTES, "rows of the four wavefronts fit the rings");
        char* const mine = smem + wave * 64 * OPITCH;                 // this wavefront's rows only: no barrier
        const TensorView& dst = role == 0 ? dV : dK;
        const float f = role == 0 ? 1.f : scale;
#pragma unroll
        for (int kg = 0; kg < 2; ++kg)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    u32x2_t wv;
                    wv.x = pack_bf16x2(acc[kg][dt][4 * g + 0] * f, acc[kg][dt][4 * g + 1] * f);
                    wv.y = pack_bf16x2(acc[kg][dt][4 * g + 2] * f, acc[kg][dt][4 * g + 3] * f);
                    *reinterpret_cast<u32x2_t*>(mine + (kg * 32 + l32) * OPITCH + (dt * 32 + g * 8 + hf * 4) * 2) = wv;
                }
        char* const base = dst.ptr + ((long long)b * dst.stride_b + (long long)h * dst.stride_h) * 2 + lane % LPR * 16;
#pragma unroll
        for (int k = 0; k < LPR; ++k) {
            const int r = k * (64 / LPR) + lane / LPR;
            const u32x4_t x = *reinterpret_cast<const u32x4_t*>(mine + r * OPITCH + lane % LPR * 16);
            if (kbase + r < L) {
                const int pos = k0 + kbase + r;
                *reinterpret_cast<u32x4_t*>(base + (long long)(rows ? rows[pos] : pos) * dst.stride_s * 2) = x;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA dK/dV kernel for a block's last L % 128 keys when they are at most 32.  The pair kernel above
// spends a whole walk of the block's query list on every 128-key run, however few of its keys exist; here
// the cost follows the keys: one workgroup per (head, block), its four wavefronts hold the same <= 32 keys
// and split the query list (wavefront w takes the 32-query chunks w, w + 4, ...), each computing all four
// products for its chunks (same operand orientation as above, key = MFMA column) from its own LDS tiles,
// without workgroup barriers; the four partial dK^T / dV^T are added through LDS at the end.
template <int D>
__device__ __forceinline__ void dkv_tail_body(
    char* smem, int bh, const int4 desc, const TensorView& Q, const TensorView& K, const TensorView& V, const TensorView& dO,
    const float* __restrict__ lse_delta, const int* __restrict__ q_idx, const TensorView& dK, const TensorView& dV, const int* __restrict__ rows,
    const int* __restrict__ kv_rows, int Hh, int S, long long cap, float scale_log2, float scale) {
    constexpr int QC = 32;                       // queries per chunk
    constexpr int STR = D + 8;
    constexpr int KSTEPS = D / 16, DT = D / 32;
    constexpr int LOADS = QC * (D / 8) / 64;     // 16-byte pieces per lane per chunk and tensor
    // Q tiles, then dO tiles, one of each per wavefront; then LSE and delta
    __bf16(*sT)[4][QC * STR] = reinterpret_cast<__bf16(*)[4][QC * STR]>(smem);
    float(*sL)[QC] = reinterpret_cast<float(*)[QC]>(smem + 2 * 4 * QC * STR * 2);
    float(*sDl)[QC] = reinterpret_cast<float(*)[QC]>(smem + 2 * 4 * QC * STR * 2 + 4 * QC * 4);
    static_assert(2 * 4 * QC * STR * 2 + 2 * 4 * QC * 4 <= DkvLds<D>::BYTES, "the tail body fits the pair body's LDS");
    const int b = bh / Hh, h = bh % Hh;
    const int tail = desc.y - TAIL_SLOT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hf = lane >> 5;
    const int cnt = desc.w;
    const int* list = q_idx + (long long)bh * cap + desc.z;
    const float* lse_h = lse_delta + (long long)bh * 2 * lse_delta_pitch(S);
    const float* dl_h = lse_h + lse_delta_pitch(S);

    // the tail keys: B operands (key = lane % 32); columns past the tail repeat the block's last key and are not written
    const bool key_live = l32 < tail;
    const int krow = desc.x + min(l32, tail - 1);
    bf16x8_t kf[KSTEPS], vf[KSTEPS];
    {
        const long long kin = kv_rows ? kv_rows[krow] : krow;         // row of K and V that holds this key
        const char* pk = K.ptr + ((long long)b * K.stride_b + kin * K.stride_s + (long long)h * K.stride_h) * 2;
        const char* pv = V.ptr + ((long long)b * V.stride_b + kin * V.stride_s + (long long)h * V.stride_h) * 2;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            kf[ks] = *reinterpret_cast<const bf16x8_t*>(pk + (ks * 16 + hf * 8) * 2);
            vf[ks] = *reinterpret_cast<const bf16x8_t*>(pv + (ks * 16 + hf * 8) * 2);
        }
    }
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t dvacc[DT], dkacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) { dvacc[dt] = zero16; dkacc[dt] = zero16; }

    const char* qbase = Q.ptr + ((long long)b * Q.stride_b + (long long)h * Q.stride_h) * 2;
    const char* dobase = dO.ptr + ((long long)b * dO.stride_b + (long long)h * dO.stride_h) * 2;
    const long long qss = Q.stride_s * 2, doss = dO.stride_s * 2;
    const int n_chunks = (cnt + QC - 1) / QC;
    __bf16* tQ = &sT[0][wave][0];
    __bf16* tdO = &sT[1][wave][0];
    float* tL = &sL[wave][0];
    float* tDl = &sDl[wave][0];
    // LSE / delta of row r are stored at the place where the accumulator layout wants them: a lane half reads its 16 rows
    // (acc_row(i, hf), i = 0..15) as 16 consecutive floats
    const int ld_pos = ((l32 & 1) << 4) + ((l32 >> 4) << 3) + (((l32 >> 1) & 1) << 2) + ((l32 >> 2) & 3);
    const int row_lane = rho(l32) * STR + hf * 8;
    const int tr_lane = tr_lane_offset<STR>(lane);

    // Gathered rows travel list index -> row address -> registers -> LDS; a wavefront keeps the rows of its next two
    // chunks in flight (register sets 0 / 1 by chunk parity) and the list indices of the one after.
    struct RowSet {
        u32x4_t q[LOADS], d[LOADS];
        float l, dl;
        bool live;
    };
    RowSet rs[2];
    int qn[LOADS], ql = 0;
    bool ql_live = false;
    auto fetch_idx = [&](int c) {                // list entries of chunk c (entries past the list repeat its last one)
        const int c0 = c * QC;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) qn[i] = list[max(min(c0 + (lane + 64 * i) / (D / 8), cnt - 1), 0)];
        ql = list[max(min(c0 + l32, cnt - 1), 0)];
        ql_live = c0 + l32 < cnt;
    };
    auto fetch_rows = [&](RowSet& r) {           // rows of the chunk whose indices were fetched last
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int pc = (lane + 64 * i) % (D / 8);
            r.q[i] = *reinterpret_cast<const u32x4_t*>(qbase + (long long)qn[i] * qss + pc * 16);
            r.d[i] = *reinterpret_cast<const u32x4_t*>(dobase + (long long)qn[i] * doss + pc * 16);
        }
        r.l = lse_h[ql];
        r.dl = dl_h[ql];
        r.live = ql_live;
    };
    auto stage = [&](const RowSet& r) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int piece = lane + 64 * i;
            const int row = piece / (D / 8), pc = piece % (D / 8);
            *reinterpret_cast<u32x4_t*>(&tQ[row * STR + pc * 8]) = r.q[i];
            *reinterpret_cast<u32x4_t*>(&tdO[row * STR + pc * 8]) = r.d[i];
        }
        if (hf == 0) {                           // rows past the end of the list: LSE = +inf (weight 0), delta = 0
            tL[ld_pos] = r.live ? r.l : INFINITY;
            tDl[ld_pos] = r.live ? r.dl : 0.f;
        }
    };
    // the wavefront's k-th chunk is chunk wave + 4 k
    const int my_chunks = n_chunks > wave ? (n_chunks - wave + 3) / 4 : 0;
    if (my_chunks > 0) {
        fetch_idx(wave);
        fetch_rows(rs[0]);
        fetch_idx(wave + 4);
        fetch_rows(rs[1]);
        fetch_idx(wave + 8);
    }
    auto one_chunk = [&](int k, RowSet& r) {
        stage(r);
        fetch_rows(r);                           // chunk k + 2 (indices are already here)
        fetch_idx(wave + 4 * (k + 3));
        // S = Q . K^T and dP = dO . V^T
        f32x16_t sacc = zero16, dpacc = zero16;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const bf16x8_t qa = *reinterpret_cast<const bf16x8_t*>(tQ + row_lane + ks * 16);
            const bf16x8_t da = *reinterpret_cast<const bf16x8_t*>(tdO + row_lane + ks * 16);
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa, kf[ks], sacc, 0, 0, 0);
            dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da, vf[ks], dpacc, 0, 0, 0);
        }
        float ld[16], dl[16];
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4_t a4 = *reinterpret_cast<const f32x4_t*>(tL + hf * 16 + g4 * 4);
            const f32x4_t d4 = *reinterpret_cast<const f32x4_t*>(tDl + hf * 16 + g4 * 4);
#pragma unroll
            for (int u = 0; u < 4; ++u) { ld[g4 * 4 + u] = a4[u]; dl[g4 * 4 + u] = d4[u]; }
        }
        float pw[16], dsw[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            pw[i] = exp2_raw(fmaf(sacc[i], scale_log2, -ld[i]));
            dsw[i] = pw[i] * (dpacc[i] + dl[i]);
        }
        // dV^T += dO^T . P and dK^T += Q^T . dS
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const bf16x8_t pb = pack8(&pw[8 * s2]);
            const bf16x8_t db = pack8(&dsw[8 * s2]);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const bf16x8_t dot = tr_operand<STR>(tdO + tr_lane, 0, s2, dt * 32);
                const bf16x8_t qt = tr_operand<STR>(tQ + tr_lane, 0, s2, dt * 32);
                dvacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dot, pb, dvacc[dt], 0, 0, 0);
                dkacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qt, db, dkacc[dt], 0, 0, 0);
            }
        }
    };
    for (int k = 0; k < my_chunks; k += 2) {
        one_chunk(k, rs[0]);
        if (k + 1 < my_chunks) one_chunk(k + 1, rs[1]);
    }
    // ---- add the four wavefronts' partial sums (the row tiles are free now) and write the tail's rows
    static_assert(2 * 4 * QC * STR * 2 >= 3 * 64 * DT * 16 * sizeof(float), "reduction buffer fits the row tiles");
    float* red = reinterpret_cast<float*>(&sT[0][0][0]);       // [3][DT * 16][64]
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        f32x16_t* acc = pass == 0 ? dvacc : dkacc;
        __syncthreads();
        if (wave > 0) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) red[((wave - 1) * DT * 16 + dt * 16 + i) * 64 + lane] = acc[dt][i];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int w = 0; w < 3; ++w)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[dt][i] += red[(w * DT * 16 + dt * 16 + i) * 64 + lane];
            if (key_live) {
                const TensorView& dst = pass == 0 ? dV : dK;
                const float fsc = pass == 0 ? 1.f : scale;
                const int kout = rows ? rows[krow] : krow;
                char* pd = dst.ptr + ((long long)b * dst.stride_b + (long long)kout * dst.stride_s + (long long)h * dst.stride_h) * 2;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        u32x2_t wv;
                        wv.x = pack_bf16x2(acc[dt][4 * g + 0] * fsc, acc[dt][4 * g + 1] * fsc);
                        wv.y = pack_bf16x2(acc[dt][4 * g + 2] * fsc, acc[dt][4 * g + 3] * fsc);
                        *reinterpret_cast<u32x2_t*>(pd + (dt * 32 + g * 8 + hf * 4) * 2) = wv;
                    }
            }
        }
    }
}

// The dK/dV launch.  Every head has `slots` slots: slots [0, runs of the head) run the pair body on one 128-key run each
// (longest query list first); the next n_blocks slots run the tail body on one block each; the rest do nothing.  Slots
// are handed out slot group first, head second (see the kernel): the order is longest-first over the whole launch
// rather than per head, and the short tail workgroups fill its end, where the long runs finish unevenly.
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_dkv_kernel(
    TensorView Q, TensorView K, TensorView V, TensorView dO, const float* __restrict__ lse_delta, const int* __restrict__ q_idx,
    const int4* __restrict__ slot_desc, TensorView dK, TensorView dV, const int* __restrict__ rows, int Hh, int S, long long cap,
    float scale_log2, float scale, const int* __restrict__ kv_rows, int BH, int slots, int group) {
    __shared__ __align__(16) char smem[DkvLds<D>::BYTES];
    // One-dimensional grid.  Workgroup i runs on XCD i % 8 as that XCD's workgroup number i / 8.  A head's slots are cut
    // into groups of `group` consecutive slots (the runs of one key block, when the blocks are equally long); groups are
    // numbered slot group first, head second -- longest query lists first over the whole launch -- and dealt to the XCDs
    // in turn, each XCD taking the slots of a group one after the other: the runs of one block, which all walk the same
    // query list, run at the same time on the same XCD and share its L2.
    const int xcd = (int)blockIdx.x & 7, n = (int)blockIdx.x >> 3;
    const int G = (n / group) * 8 + xcd;
    if (G >= BH * (slots / group)) return;
    const int bh = G % BH;
    const int id = (G / BH) * group + n % group;
    const int4 desc = slot_desc[(long long)bh * slots + id];
    if (desc.y == 0) return;
    if (desc.y < TAIL_SLOT)
        dkv_pair_body<D>(smem, bh, desc, Q, K, V, dO, lse_delta, q_idx, dK, dV, rows, kv_rows, Hh, S, cap, scale_log2, scale);
    else
        dkv_tail_body<D>(smem, bh, desc, Q, K, V, dO, lse_delta, q_idx, dK, dV, rows, kv_rows, Hh, S, cap, scale_log2, scale);
}

// dQ[q] = scale * sum over the query's pairs of dQpart[pair]; the partials have the tensors' type.  A head whose
// selection did not fit the lists (row_ptr[S] > cap, see vmoba_select) counts as having selected nothing.
template <bool BF16, int D>
__global__ __launch_bounds__(256) void dq_merge_kernel(const float* __restrict__ dQpart, const int* __restrict__ row_ptr,
                                                       const int* __restrict__ pair_pos, TensorView dQ, const int* __restrict__ rows, int Hh, int S,
                                                       long long cap, float scale) {
    constexpr int CH = BF16 ? 8 : 4;
    constexpr int LPQ = D / CH;
    constexpr int QPW = 256 / LPQ;
    const int bh = blockIdx.y, b = bh / Hh, h = bh % Hh;
    const int q = blockIdx.x * QPW + threadIdx.x / LPQ;
    const int part = threadIdx.x % LPQ;
    if (q >= S) return;
    const bool fits = row_ptr[(long long)bh * (S + 1) + S] <= cap;
    const int r0 = row_ptr[(long long)bh * (S + 1) + q];
    const int r1 = fits ? row_ptr[(long long)bh * (S + 1) + q + 1] : r0;
    const long long seg = (long long)bh * cap;
    float acc[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[c] = 0.f;
    constexpr int MB = 8;                            // partial rows in flight per lane
    for (int r = r0; r < r1; r += MB) {
        long long pair[MB];
#pragma unroll
        for (int u = 0; u < MB; ++u) pair[u] = seg + pair_pos[seg + min(r + u, r1 - 1)];
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const float keep = (r + u < r1) ? 1.f : 0.f;
            if constexpr (BF16) {
                // (read once: non-temporal, as in the forward merge)
                const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(dQpart) + pair[u] * D + part * 8));
                acc[0] += keep * bf16lo_to_f32(v.x); acc[1] += keep * bf16hi_to_f32(v.x);
                acc[2] += keep * bf16lo_to_f32(v.y); acc[3] += keep * bf16hi_to_f32(v.y);
                acc[4] += keep * bf16lo_to_f32(v.z); acc[5] += keep * bf16hi_to_f32(v.z);
                acc[6] += keep * bf16lo_to_f32(v.w); acc[7] += keep * bf16hi_to_f32(v.w);
            } else {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(dQpart + pair[u] * D + part * 4);
                acc[0] += keep * v.x; acc[1] += keep * v.y; acc[2] += keep * v.z; acc[3] += keep * v.w;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[c] *= scale;
    const int qo = rows ? rows[q] : q;
    char* dst = dQ.ptr + ((long long)b * dQ.stride_b + (long long)qo * dQ.stride_s + (long long)h * dQ.stride_h) * (BF16 ? 2 : 4);
    if constexpr (BF16) {
        const u32x4_t o = {pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]), pack_bf16x2(acc[4], acc[5]),
                           pack_bf16x2(acc[6], acc[7])};
        *reinterpret_cast<u32x4_t*>(dst + part * 16) = o;
    } else {
#pragma unroll
        for (int c = 0; c < CH; c += 4) {
            f32x4_t o = {acc[c], acc[c + 1], acc[c + 2], acc[c + 3]};
            *reinterpret_cast<f32x4_t*>(dst + (part * CH + c) * 4) = o;
        }
    }
}

struct BwdWs {
    float* dQpart;     // [BH * cap][D], in the tensors' type
    float* delta;      // LSE * log2(e) and -delta, [BH][2][lse_delta_pitch(S)]
    int* n_tiles;      // length of the tile list, then the split kernels' flag
    int* head_tiles;   // [BH]
    int4* tile_desc;   // the flat list of all heads' tiles
    int* kb_start;     // float32: [BH][nb + 1]
    int* kb_order;     // float32: [BH][nb]
    int4* slot_desc;   // bfloat16: [BH][dkv_slots]
    char* dO_copy;     // [BH, S, D] block-order copy of dO (used with a row map)
    char* QD6;         // split kernels: [BH][S][6][D], the terms of Q and dO by query id, and those of K and V in block order (see attn_split.hip)
    char* KV6;
    size_t total;
};

// Slots of the matrix-core dK/dV kernels per head: `group` consecutive ones are one block's runs (the usual block: S / nb keys; bfloat16:
// a last run of at most 32 keys goes to the tail workgroups); in all a multiple of group and of 8 (workgroup id % 8 is then the same for every
// head), + 8 for the per-XCD rounding.
struct DkvSlots { int grid_x, group, slots; };
DkvSlots dkv_slots(int64_t S, int nb, int KPW, bool bf16) {
    const int64_t usual = S / nb;
    DkvSlots d;
    d.grid_x = (int)((S / KPW + nb + 7) / 8 * 8 + 8 + (bf16 ? nb : 0));
    d.group = (int)std::max<int64_t>(1, (bf16 && usual % KPW > 0 && usual % KPW <= 32) ? usual / KPW : ceil_div64(usual, KPW));
    d.slots = (int)ceil_div64(d.grid_x, d.group) * d.group;
    return d;
}

constexpr int BWD_TM = 128;                   // queries per dQ tile

BwdWs carve_bwd(void* base, int BH, int64_t S, int D, int nb, int64_t cap, int es, bool split) {
    BwdWs w;
    char* p = (char*)base;
    size_t off = 0;
    w.dQpart = (float*)(p + off);    off += align_up((size_t)BH * cap * D * es, 256);
    w.delta = (float*)(p + off);     off += align_up((size_t)BH * 2 * (size_t)lse_delta_pitch((int)S) * 4, 256);
    w.n_tiles = (int*)(p + off);     off += 256;
    w.head_tiles = (int*)(p + off);  off += align_up((size_t)BH * 4, 256);
    // The tile list and what the dK/dV kernels find their work by.  The slots of a bfloat16 call lie behind the tiles that there can be and in the
    // place of the float32 kernels' arrays, so that they need scratch of their own only for calls of many blocks and few pairs.
    w.tile_desc = (int4*)(p + off);
    const size_t list = align_up((size_t)BH * vmoba_max_tiles(cap, 64) * 16, 256), start = align_up((size_t)BH * (VMOBA_MAX_BLOCKS + 1) * 4, 256),
                 order = align_up((size_t)BH * VMOBA_MAX_BLOCKS * 4, 256);
    w.kb_start = (int*)(p + off + list);
    w.kb_order = (int*)(p + off + list + start);
    const size_t tiles = align_up((size_t)BH * (cap / BWD_TM + nb) * 16, 256);
    w.slot_desc = (int4*)(p + off + tiles);
    off += list + start + order;
    if (es == 2) off = std::max(off, (size_t)((char*)w.slot_desc - p) + align_up((size_t)BH * dkv_slots(S, nb, 128, true).slots * 16, 256));
    w.dO_copy = p + off;             off += align_up((size_t)BH * S * D * es, 256);
    w.QD6 = p + off;                 off += split ? align_up((size_t)BH * S * 12 * D, 256) : 0;
    w.KV6 = p + off;                 off += split ? align_up((size_t)BH * S * 12 * D, 256) : 0;
    w.total = off;
    return w;
}

}  // namespace

size_t vmoba_attn_bwd_workspace_bytes(int B, int Hh, int64_t S, int D, int nb, int64_t cap, int dtype) {
    const bool bf16 = dtype == VMOBA_BF16;
    return carve_bwd(nullptr, B * Hh, S, D, nb, cap, bf16 ? 2 : 4, !bf16 && use_split(B * Hh, S, D, nb, cap)).total;
}

extern "C" int vmoba_attn_bwd(int B, int Hh, int64_t S, int D, int32_t n_blocks, const int32_t* blk_off,
                              const vmoba_tensor* Qp, const vmoba_tensor* Kp, const vmoba_tensor* Vp,
                              const vmoba_tensor* O, const float* LSE, const vmoba_tensor* dO,
                              const int32_t* blk_ptr, const int32_t* q_idx, const int32_t* row_ptr,
                              const int32_t* pair_pos, int64_t nnz_capacity, float softmax_scale,
                              const vmoba_tensor* dQ, const vmoba_tensor* dK, const vmoba_tensor* dV,
                              const int32_t* rows, const int32_t* key_rows, const int32_t* kv_rows, void* workspace,
                              size_t workspace_bytes, void* stream) {
    if (B <= 0 || Hh <= 0 || S <= 0 || n_blocks <= 0 || nnz_capacity <= 0) return VMOBA_ERR_INVALID_ARG;
    if (!blk_off || !blk_ptr || !q_idx || !row_ptr || !pair_pos || !LSE || !workspace) return VMOBA_ERR_INVALID_ARG;
    if (!tensor_ok(Qp) || !tensor_ok(Kp) || !tensor_ok(Vp) || !tensor_ok(O) || !tensor_ok(dO) || !tensor_ok(dQ) ||
        !tensor_ok(dK) || !tensor_ok(dV))
        return VMOBA_ERR_INVALID_ARG;
    if (!std::isfinite(softmax_scale)) return VMOBA_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return VMOBA_ERR_UNSUPPORTED;
    if (n_blocks > VMOBA_MAX_BLOCKS) return VMOBA_ERR_UNSUPPORTED;
    const int dt = Qp->dtype;
    if (Kp->dtype != dt || Vp->dtype != dt || O->dtype != dt || dO->dtype != dt || dQ->dtype != dt ||
        dK->dtype != dt || dV->dtype != dt)
        return VMOBA_ERR_UNSUPPORTED;
    const int BH = B * Hh;
    if (nnz_capacity > INT32_MAX) return VMOBA_ERR_UNSUPPORTED;
    const bool bf16 = dt == VMOBA_BF16;
    const bool split = !bf16 && use_split(BH, S, D, n_blocks, nnz_capacity);
    BwdWs ws = carve_bwd(workspace, BH, S, D, n_blocks, nnz_capacity, bf16 ? 2 : 4, split);
    if (workspace_bytes < ws.total) return VMOBA_ERR_WORKSPACE;
    if (((uintptr_t)workspace) & 255) return VMOBA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const TensorView Qv = make_view(Qp), Kv = make_view(Kp), Vv = make_view(Vp), Ov = make_view(O);
    const TensorView dQv = make_view(dQ), dKv = make_view(dK), dVv = make_view(dV);
    TensorView dOv = make_view(dO);
    const float scale_log2 = softmax_scale * LOG2E;
    // the bfloat16 kernels form the byte offset of a row of Q', K', V' or dO with one 24-bit multiply and 32-bit adds
    if (bf16) {
        const int64_t do_stride = rows ? D : dO->stride_s;          // dO is read from its block-order copy when `rows` is given
        const int64_t strides[4] = {Qp->stride_s, Kp->stride_s, Vp->stride_s, do_stride};
        if (S >= (1 << 24)) return VMOBA_ERR_UNSUPPORTED;
        for (int64_t ss : strides)
            if (ss <= 0 || ss * 2 >= (1 << 24) || (uint64_t)S * (uint64_t)ss * 2 >= ((uint64_t)1 << 32)) return VMOBA_ERR_UNSUPPORTED;
    }

    // ---- delta, tile list, key runs
    const int TM = BWD_TM;
    int* const out_of_range = ws.n_tiles + 1;
    const int KPW = bf16 || split ? 128 : 64;        // keys per dK/dV workgroup
    const DkvSlots dkv = dkv_slots(S, n_blocks, KPW, bf16);
    const int64_t max_tiles = std::min<int64_t>(vmoba_max_tiles(nnz_capacity, TM), (nnz_capacity / TM + n_blocks + 7) / 8 * 8);
    {
        const int* head_tiles = heads_counted_first(BH, n_blocks) ? ws.head_tiles : nullptr;
        if (head_tiles) launch_head_tiles(st, blk_ptr, ws.head_tiles, BH, n_blocks, TM);
        const int n_delta = (int)ceil_div64(S, 256 / (D / (bf16 ? 8 : 4)));
        const dim3 grid((unsigned)(n_delta + ceil_div64(max_tiles, 256) + 1), (unsigned)BH);
        auto kfn = bf16 ? (D == 128 ? bwd_prepare_kernel<true, 128> : bwd_prepare_kernel<true, 64>)
                        : (D == 128 ? bwd_prepare_kernel<false, 128> : bwd_prepare_kernel<false, 64>);
        kfn<<<grid, dim3(256), 0, st>>>(Ov, dOv, LSE, ws.delta, rows, ws.dO_copy, blk_ptr, blk_off, head_tiles, ws.tile_desc, ws.n_tiles, out_of_range, ws.kb_start, ws.kb_order, ws.slot_desc, dkv.slots,
                                        BH, Hh, (int)S, n_blocks, TM, KPW, bf16 ? 32 : 0, n_delta);
        VMOBA_CHECK_LAUNCH();
    }
    if (rows) {   // from here on dO is the block-order copy [B, Hh, S, D] the delta kernel wrote
        dOv.ptr = ws.dO_copy;
        dOv.stride_b = (int64_t)Hh * S * D;
        dOv.stride_h = S * D;
        dOv.stride_s = D;
    }
    if (split) {
        launch_split_rows(D, BH, Hh, (int)S, st, Qv, nullptr, ws.QD6, 6, 0, out_of_range);
        launch_split_rows(D, BH, Hh, (int)S, st, dOv, nullptr, ws.QD6, 6, 3, out_of_range);
        launch_split_rows(D, BH, Hh, (int)S, st, Kv, kv_rows, ws.KV6, 6, 0, out_of_range);
        launch_split_rows(D, BH, Hh, (int)S, st, Vv, kv_rows, ws.KV6, 6, 3, out_of_range);
        VMOBA_CHECK_LAUNCH();
    }
    const int pitch = lse_delta_pitch((int)S);
    // ---- dQ
    {
        VMOBA_PROFILE_BEGIN(1, st);
        const dim3 grid = flat_tile_grid(BH, max_tiles, nnz_capacity, TM, n_blocks);     // one workgroup per tile
        if (!bf16) {
            if (split)
                launch_dq_tiles_split(D, grid, st, ws.QD6, ws.KV6, ws.delta, q_idx, ws.tile_desc, ws.n_tiles, out_of_range, ws.dQpart, (int)S, pitch,
                                      (long long)nnz_capacity, scale_log2);
            launch_dq_tiles_f32(D, grid, st, split ? out_of_range : nullptr, Qv, Kv, Vv, dOv, ws.delta, q_idx, ws.tile_desc, ws.n_tiles, ws.dQpart, Hh, (int)S,
                                (long long)nnz_capacity, scale_log2, kv_rows);
        } else {
#define DQ_ARGS Qv, Kv, Vv, dOv, ws.delta, q_idx, ws.tile_desc, ws.n_tiles, ws.dQpart, Hh, (int)S, (long long)nnz_capacity, scale_log2, kv_rows
            if (D == 128) attn_bwd_dq_mfma_kernel<128><<<grid, dim3(256), 0, st>>>(DQ_ARGS);
            else attn_bwd_dq_mfma_kernel<64><<<grid, dim3(256), 0, st>>>(DQ_ARGS);
#undef DQ_ARGS
        }
        VMOBA_PROFILE_END(1, st);
        VMOBA_CHECK_LAUNCH();
        const int qpw = 256 / (D / (bf16 ? 8 : 4));     // partials in the tensors' type
        dim3 mgrid((unsigned)ceil_div64(S, qpw), (unsigned)BH);
#define MG_ARGS ws.dQpart, row_ptr, pair_pos, dQv, rows, Hh, (int)S, (long long)nnz_capacity, softmax_scale
        if (bf16 && D == 128) dq_merge_kernel<true, 128><<<mgrid, dim3(256), 0, st>>>(MG_ARGS);
        else if (bf16) dq_merge_kernel<true, 64><<<mgrid, dim3(256), 0, st>>>(MG_ARGS);
        else if (D == 128) dq_merge_kernel<false, 128><<<mgrid, dim3(256), 0, st>>>(MG_ARGS);
        else dq_merge_kernel<false, 64><<<mgrid, dim3(256), 0, st>>>(MG_ARGS);
#undef MG_ARGS
        VMOBA_CHECK_LAUNCH();
    }
    // ---- dK, dV
    {
        const dim3 hgrid((unsigned)(ceil_div64((int64_t)BH * dkv.slots, 8) * 8 + 7 * dkv.group));   // see the kernel
        VMOBA_PROFILE_BEGIN(2, st);
        const int32_t* krows = key_rows ? key_rows : rows;      // row map of dK and dV
#define DKV_ARGS blk_off, blk_ptr, q_idx, ws.kb_start, ws.kb_order, dKv, dVv, krows, Hh, (int)S, n_blocks, (long long)nnz_capacity, scale_log2, softmax_scale, kv_rows
        if (!bf16) {
            if (split)
                launch_dkv_split(D, hgrid, st, ws.QD6, ws.KV6, ws.delta, blk_off, blk_ptr, q_idx, ws.kb_start, ws.kb_order, out_of_range, dKv, dVv, krows,
                                 Hh, (int)S, pitch, n_blocks, (long long)nnz_capacity, scale_log2, softmax_scale, BH, dkv.slots, dkv.group);
            const int parts = split ? 2 : 1;
            launch_dkv_f32(D, dim3((unsigned)(dkv.grid_x * parts), (unsigned)BH), st, split ? out_of_range : nullptr, parts, Qv, Kv, Vv, dOv, ws.delta, DKV_ARGS);
        } else {
            auto kfn = D == 128 ? attn_bwd_dkv_kernel<128> : attn_bwd_dkv_kernel<64>;
            kfn<<<hgrid, dim3(256), 0, st>>>(Qv, Kv, Vv, dOv, ws.delta, q_idx, ws.slot_desc, dKv, dVv, krows, Hh, (int)S, (long long)nnz_capacity,
                                             scale_log2, softmax_scale, kv_rows, BH, dkv.slots, dkv.group);
        }
#undef DKV_ARGS
        VMOBA_PROFILE_END(2, st);
        VMOBA_CHECK_LAUNCH();
    }
    return VMOBA_OK;
}
