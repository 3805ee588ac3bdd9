// Block-sparse attention kernels for float32 tensors, forward and backward, on the float32 matrix instruction
// v_mfma_f32_32x32x2_f32 (every product and sum in float32; 64 cycles for 4096 FLOP, 157 TFLOP/s on the whole chip).
//
// For the calls that the kernels on split operands (attn_split.hip) do not take: small ones (use_split), and those whose tensors hold
// infinities, NaNs or magnitudes out of the range that three bfloat16 terms hold.
//
// Work decomposition as in the bfloat16 kernels: a tile is up to 128 gathered queries of one key block (forward, dQ), a
// run is up to 64 keys of one block that meet the block's whole query list (dK/dV).
//
// What bounds them: the matrix pipe.  A 32 x 32 piece of S is D / 2 instructions of 64 cycles, its soft-max about 100
// vector instructions in all, and an operand is one 4-byte value per lane (a 16-byte LDS read serves four instructions),
// so neither the vector unit nor the LDS is near its limit and no software pipeline inside the wavefront is needed.
//
// Operand plumbing (lane = 32*hf + l32).  A: row l32, contraction index hf.  B: column l32, contraction index hf.
// C/D: column l32, row 8*i + 4*hf + r as value 4*i + r.  A contraction index may be named freely as long as A and B
// agree, so
//   * products over channels take channel 8*g + 4*hf + m in instruction 4*g + m: both operands are 16-byte pieces;
//   * products over the rows of S take row 8*i + 4*hf + r in instruction 4*i + r: the B operand is accumulator value
//     4*i + r itself, with no shuffle and no conversion, the A operand a 4-byte read of that row of the LDS tile.
//
// Measured on 14 040 tokens x 12 heads x 128 (36 blocks of 390 keys, 785 K kept pairs): forward 1.45 ms (109 TFLOP/s), dQ
// 2.32 ms (102), dK/dV 3.34 ms (94, the last run of a block holds 6 keys of 64); the plain FMA kernels before took 15.3,
// 15.4 and 72 ms (a query or key per lane: one LDS broadcast read per four FMAs, and 512 registers with spills in dK/dV).  That call
// comes here only when its operands are out of the other kernels' range; the smallest layers are bound by their launches.
// A dense product on the same instruction reaches 153 TFLOP/s.
//
// Rows travel from global memory straight to LDS (16 bytes per lane), one chunk ahead in a second buffer, one barrier per
// chunk.  16-byte piece p of tile row r sits at piece position p ^ (r % pieces per row): row reads spread over all banks
// and the 4-byte reads of 32 consecutive channels of a row stay inside one 128-byte run.
#include "attn_common.h"

namespace {

constexpr float LN2 = 0.6931471805599453f;

// 64 lanes x 16 (4) bytes from a 64-bit address per lane to LDS: lane i writes lds_addr + 16 (4) * i.
__device__ __forceinline__ void dma16_at(const char* src, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}
__device__ __forceinline__ void dma4_at(const char* src, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_address(const char* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ f32x16_t mfma2(float a, float b, f32x16_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// Reads of a 32-row tile as the kernels above describe them.
template <int D>
struct TileReads {
    static constexpr int RB = 4 * D, PPR = RB / 16;      // bytes and 16-byte pieces per row
    uint32_t row_off;                                    // row l32, piece hf (swizzled); piece 2*g + hf: XOR with g << 5
    uint32_t col_off[4];                                 // row 4*hf + r, channel l32 (swizzled)
    __device__ __forceinline__ TileReads(int lane) {
        const int l32 = lane & 31, hf = lane >> 5;
        row_off = (uint32_t)(l32 * RB + ((hf ^ l32) & (PPR - 1)) * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            col_off[r] = (uint32_t)((4 * hf + r) * RB + (((l32 >> 2) ^ (4 * hf) ^ r) & 7) * 16 + (l32 & 3) * 4);
    }
    // channels 8*g + 4*hf .. + 3 of row l32
    __device__ __forceinline__ f32x4_t rows(const char* tile, int g) const {
        return *reinterpret_cast<const f32x4_t*>(tile + (row_off ^ (uint32_t)(g << 5)));
    }
    // channel 32*dt + l32 of row 8*i + 4*hf + r (the row's bits 3 and 4 meet those of the channel's piece)
    __device__ __forceinline__ float cols(const char* tile, int i, int r, int dt) const {
        return *reinterpret_cast<const float*>(tile + col_off[r] + (8 * i * RB + (((8 * dt) ^ (8 * i)) & (PPR - 1)) * 16));
    }
};

// One wavefront's share of the K and V rows of a tile's 32-key chunks.  The rows that hold a chunk's keys -- the key
// positions themselves, or what kv_rows says -- are looked up one chunk before they are requested, so that a request never
// waits for its lookup.  Keys past the block's end repeat its last one.
template <int D>
struct KeyRows {
    static constexpr int RB = 4 * D, PPR = RB / 16, RPI = 1024 / RB, TILE = 32 * RB, IPW = TILE / 1024 / 4;
    const char* kbase;
    const char* vbase;
    long long kss, vss;                                  // row strides in bytes
    const int* kv_rows;
    int k0, L, lane, wave;
    int row[IPW];
    __device__ __forceinline__ void look_up(int c) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const int pos = k0 + min(c * 32 + (wave * IPW + i) * RPI + lane / PPR, L - 1);
            row[i] = kv_rows ? kv_rows[pos] : pos;
        }
    }
    __device__ __forceinline__ void request(uint32_t k_tile, uint32_t v_tile) const {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const int n = wave * IPW + i, r = n * RPI + lane / PPR;
            const int piece = ((lane % PPR) ^ (r & (PPR - 1))) * 16;
            dma16_at(kbase + row[i] * kss + piece, k_tile + (uint32_t)n * 1024);
            dma16_at(vbase + row[i] * vss + piece, v_tile + (uint32_t)n * 1024);
        }
    }
};

// Registers <- the channels of one row that a lane half holds (B operand of the products over channels).
template <int D>
__device__ __forceinline__ void load_row_half(const char* src, int hf, float (&dst)[D / 2]) {
#pragma unroll
    for (int g = 0; g < D / 8; ++g) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(src + (8 * g + 4 * hf) * 4);
        dst[4 * g] = v.x; dst[4 * g + 1] = v.y; dst[4 * g + 2] = v.z; dst[4 * g + 3] = v.w;
    }
}

// Products over channels, one or two side by side: step g reads the operands of g + 1, then multiplies those of g.
template <int D>
__device__ __forceinline__ void product_over_channels(const TileReads<D>& rd, const char* ta, const float (&fa)[D / 2], f32x16_t& sa) {
    f32x4_t a = rd.rows(ta, 0);
#pragma unroll
    for (int g = 0; g < D / 8; ++g) {
        f32x4_t an = a;
        if (g + 1 < D / 8) an = rd.rows(ta, g + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 4; ++m) sa = mfma2(a[m], fa[4 * g + m], sa);
        __builtin_amdgcn_sched_barrier(0);
        a = an;
    }
}
template <int D>
__device__ __forceinline__ void two_products_over_channels(const TileReads<D>& rd, const char* ta, const char* tb, const float (&fa)[D / 2],
                                                           const float (&fb)[D / 2], f32x16_t& sa, f32x16_t& sb) {
    f32x4_t a = rd.rows(ta, 0), b = rd.rows(tb, 0);
#pragma unroll
    for (int g = 0; g < D / 8; ++g) {
        f32x4_t an = a, bn = b;
        if (g + 1 < D / 8) { an = rd.rows(ta, g + 1); bn = rd.rows(tb, g + 1); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            sa = mfma2(a[m], fa[4 * g + m], sa);
            sb = mfma2(b[m], fb[4 * g + m], sb);
        }
        __builtin_amdgcn_sched_barrier(0);
        a = an;
        b = bn;
    }
}
// Operands of row step n of a product over the tile's rows: row 8*(n >> 2) + 4*hf + (n & 3), every channel tile.
template <int D>
__device__ __forceinline__ void read_cols(const TileReads<D>& rd, const char* tile, int n, float (&dst)[D / 32]) {
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) dst[dt] = rd.cols(tile, n >> 2, n & 3, dt);
}
// acc^T[channel, column] += tile^T . w over the tile's 32 rows; `a` holds the operands of row step 0 already.
template <int D>
__device__ __forceinline__ void product_over_rows(const TileReads<D>& rd, const char* tile, float (&a)[D / 32], const f32x16_t& w, f32x16_t (&acc)[D / 32]) {
#pragma unroll
    for (int n = 0; n < 16; ++n) {
        float an[D / 32];
        read_cols<D>(rd, tile, n + 1 < 16 ? n + 1 : n, an);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) acc[dt] = mfma2(a[dt], w[n], acc[dt]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) a[dt] = an[dt];
    }
}

__device__ __forceinline__ const char* head_ptr(const TensorView& t, int b, int h) {
    return t.ptr + ((long long)b * t.stride_b + (long long)h * t.stride_h) * 4;
}

// ---------------------------------------------------------------------------------------------
// Forward: S^T = K . Q^T, online soft-max (query on the lane), O^T += V^T . P^T.
template <int D>
__global__ __launch_bounds__(256, 2) void attn_fwd_tile_f32_kernel(
    const int* __restrict__ run_if, TensorView Q, TensorView K, TensorView V, const int* __restrict__ q_idx, const int4* __restrict__ flat_desc,
    const int* __restrict__ n_tiles, float* __restrict__ Opart, float* __restrict__ lse_part, int Hh,
    long long cap, float scale_log2, const int* __restrict__ kv_rows) {
    constexpr int KC = 32, TILE = KeyRows<D>::TILE, DT = D / 32;
    __shared__ __align__(1024) char sKV[2][2][TILE];              // [buffer][K, V]
    Tile t;
    if (run_if && !*run_if) return;
    if (!take_tile(flat_desc, n_tiles, t)) return;
    const int b = t.bh / Hh, h = t.bh % Hh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long seg = (long long)t.bh * cap;
    const int ent = wave * 32 + l32;
    const int q = q_idx[seg + t.list0 + min(ent, t.count - 1)];   // surplus rows repeat the tile's last query
    KeyRows<D> kr{head_ptr(K, b, h), head_ptr(V, b, h), K.stride_s * 4, V.stride_s * 4, kv_rows, t.k0, t.L, lane, wave};
    kr.look_up(0);
    kr.request(lds_address(sKV[0][0]), lds_address(sKV[0][1]));
    kr.look_up(1);
    float qf[D / 2];
    load_row_half<D>(head_ptr(Q, b, h) + (long long)q * Q.stride_s * 4, hf, qf);
    const TileReads<D> rd(lane);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16;
    float m_run = -INFINITY, l_run = 0.f;                         // l_run: this lane half's share of the row sum
    const int n_chunks = (t.L + KC - 1) / KC;
    for (int c = 0; c < n_chunks; ++c) {
        VMOBA_WAIT_VMCNT(0);
        __syncthreads();                                          // chunk c has landed; everybody is done with chunk c - 1
        if (c + 1 < n_chunks) {
            kr.request(lds_address(sKV[(c + 1) & 1][0]), lds_address(sKV[(c + 1) & 1][1]));
            kr.look_up(c + 2);
        }
        const char* sK = sKV[c & 1][0];
        const char* sV = sKV[c & 1][1];
        f32x16_t s = zero16;
        product_over_channels<D>(rd, sK, qf, s);
        float va[DT];
        read_cols<D>(rd, sV, 0, va);
        const int left = t.L - c * KC - 4 * hf;                   // value 4*i + r is key 8*i + r of this lane half
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] *= scale_log2;          // (a scale of any sign: scaled before the maximum)
        if (left < KC) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + (v & 3) >= left) s[v] = -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = swap_halves_max(mx);
        const float m_new = fmaxf(m_run, mx);
        if (__builtin_amdgcn_ballot_w64(m_new > m_run)) {
            const float alpha = exp2_raw(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[dt][v] *= alpha;
            m_run = m_new;
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = exp2_raw(s[v] - m_run);
            l_run += s[v];
        }
        product_over_rows<D>(rd, sV, va, s, acc);
    }
    const float l_tot = swap_halves_sum(l_run);
    if (ent < t.count) {
        const long long pair = seg + t.list0 + ent;
        const float inv = 1.f / l_tot;
        float* dst = Opart + pair * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t o = {acc[dt][4 * i] * inv, acc[dt][4 * i + 1] * inv, acc[dt][4 * i + 2] * inv, acc[dt][4 * i + 3] * inv};
                *reinterpret_cast<f32x4_t*>(dst + dt * 32 + i * 8 + hf * 4) = o;
            }
        if (hf == 0) lse_part[pair] = (m_run + log2f(l_tot)) * LN2;
    }
}

// ---------------------------------------------------------------------------------------------
// dQ: S^T = K . Q^T and dP^T = V . dO^T side by side, dS^T = P^T * (dP^T - delta), dQ^T += K^T . dS^T.
// The fragments of Q and dO and the accumulators take 192 registers: one wavefront per SIMD.
template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_dq_f32_kernel(
    const int* __restrict__ run_if, TensorView Q, TensorView K, TensorView V, TensorView dO, const float* __restrict__ lse_delta,
    const int* __restrict__ q_idx, const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles,
    float* __restrict__ dQpart, int Hh, int S, long long cap, float scale_log2, const int* __restrict__ kv_rows) {
    constexpr int KC = 32, TILE = KeyRows<D>::TILE, DT = D / 32;
    __shared__ __align__(1024) char sKV[2][2][TILE];
    Tile t;
    if (run_if && !*run_if) return;
    if (!take_tile(flat_desc, n_tiles, t)) return;
    const int b = t.bh / Hh, h = t.bh % Hh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long seg = (long long)t.bh * cap;
    const int ent = wave * 32 + l32;
    const int q = q_idx[seg + t.list0 + min(ent, t.count - 1)];
    KeyRows<D> kr{head_ptr(K, b, h), head_ptr(V, b, h), K.stride_s * 4, V.stride_s * 4, kv_rows, t.k0, t.L, lane, wave};
    kr.look_up(0);
    kr.request(lds_address(sKV[0][0]), lds_address(sKV[0][1]));
    kr.look_up(1);
    float qf[D / 2], dof[D / 2];
    load_row_half<D>(head_ptr(Q, b, h) + (long long)q * Q.stride_s * 4, hf, qf);
    load_row_half<D>(head_ptr(dO, b, h) + (long long)q * dO.stride_s * 4, hf, dof);
    const float lse2 = lse_delta[(long long)t.bh * 2 * lse_delta_pitch(S) + q];
    const float ndl = lse_delta[((long long)t.bh * 2 + 1) * lse_delta_pitch(S) + q];
    const TileReads<D> rd(lane);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16;
    const int n_chunks = (t.L + KC - 1) / KC;
    for (int c = 0; c < n_chunks; ++c) {
        VMOBA_WAIT_VMCNT(0);
        __syncthreads();
        if (c + 1 < n_chunks) {
            kr.request(lds_address(sKV[(c + 1) & 1][0]), lds_address(sKV[(c + 1) & 1][1]));
            kr.look_up(c + 2);
        }
        const char* sK = sKV[c & 1][0];
        const char* sV = sKV[c & 1][1];
        f32x16_t s = zero16, dp = zero16;
        two_products_over_channels<D>(rd, sK, sV, qf, dof, s, dp);
        float ka[DT];
        read_cols<D>(rd, sK, 0, ka);
        const int left = t.L - c * KC - 4 * hf;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = exp2_raw(fmaf(s[v], scale_log2, -lse2));
            dp[v] = p * (dp[v] + ndl);
        }
        if (left < KC) {                                          // keys past the block's end
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + (v & 3) >= left) dp[v] = 0.f;
        }
        product_over_rows<D>(rd, sK, ka, dp, acc);
    }
    if (ent < t.count) {
        float* dst = dQpart + (seg + t.list0 + ent) * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t o = {acc[dt][4 * i], acc[dt][4 * i + 1], acc[dt][4 * i + 2], acc[dt][4 * i + 3]};
                *reinterpret_cast<f32x4_t*>(dst + dt * 32 + i * 8 + hf * 4) = o;
            }
    }
}

// ---------------------------------------------------------------------------------------------
// dK/dV: a workgroup owns 64 keys of one block and walks the block's query list in chunks of 64.  Wavefront (kw, qh) =
// (wave % 2, wave / 2) holds keys 32*kw .. + 31 and meets queries 32*qh .. + 31 of every chunk (key = lane % 32):
//   S = Q . K^T,  dP = dO . V^T,  dV^T += dO^T . P,  dK^T += Q^T . dS
// The two wavefronts of a key group add their sums through LDS at the end.  64 keys rather than 128: a block's last run is
// rarely full, and the two query halves keep the LDS traffic of a shared chunk.
template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkv_f32_kernel(
    const int* __restrict__ run_if, int parts, TensorView Q, TensorView K, TensorView V, TensorView dO, const float* __restrict__ lse_delta,
    const int* __restrict__ blk_off, const int* __restrict__ blk_ptr, const int* __restrict__ q_idx,
    const int* __restrict__ kb_start, const int* __restrict__ kb_order, TensorView dK, TensorView dV, const int* __restrict__ rows, int Hh, int S, int nb, long long cap,
    float scale_log2, float scale, const int* __restrict__ kv_rows) {
    constexpr int KPW = 64, QC = 64, RB = 4 * D, HALF = 32 * RB, DT = D / 32, IPW = QC * RB / 1024 / 4, RPI = 1024 / RB, PPR = RB / 16;
    __shared__ __align__(1024) char sT[2][2][2 * HALF];           // [buffer][Q, dO]
    __shared__ float sLD[2][2][QC];                               // [buffer][LSE, -delta]
    if (run_if && !*run_if) return;
    const int run_id = (int)blockIdx.x / parts, part = (int)blockIdx.x % parts;
    const int bh = blockIdx.y, b = bh / Hh, h = bh % Hh;
    const int* ks = kb_start + (long long)bh * (nb + 1);
    if (run_id >= ks[nb]) return;
    int lo = 0, hi = nb;
    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (ks[mid] <= run_id) lo = mid; else hi = mid; }
    const int j = kb_order[(long long)bh * nb + lo];
    const int k0 = blk_off[j], L = blk_off[j + 1] - k0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5, kw = wave & 1, qh = wave >> 1;
    const int key0 = ((run_id - ks[lo]) * parts + part) * KPW;
    if (key0 >= L) return;
    const int kk = key0 + kw * 32 + l32;
    const bool live = kk < L;
    const bool wave_live = kk - l32 < L;                          // any key of this wavefront exists
    const int krow = k0 + min(kk, L - 1);
    const long long seg = (long long)bh * cap;
    const int list0 = blk_ptr[(long long)bh * (nb + 1) + j];
    const int cnt = blk_ptr[(long long)bh * (nb + 1) + j + 1] - list0;
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[2][DT];                                          // dV^T, dK^T
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[x][dt] = zero16;
    if (cnt > 0) {                                                // uniform over the workgroup
        float kf[D / 2], vf[D / 2];
        {
            const long long kin = kv_rows ? kv_rows[krow] : krow; // row of K and V that holds this key
            load_row_half<D>(head_ptr(K, b, h) + kin * K.stride_s * 4, hf, kf);
            load_row_half<D>(head_ptr(V, b, h) + kin * V.stride_s * 4, hf, vf);
        }
        const char* qbase = head_ptr(Q, b, h);
        const char* dobase = head_ptr(dO, b, h);
        const int* list = q_idx + seg + list0;
        const int n_chunks = (cnt + QC - 1) / QC;
        auto index_of = [&](int c) { return list[min(c * QC + lane, cnt - 1)]; };     // lane = row of the chunk
        auto request = [&](int c, int idx) {                      // rows past the list repeat its last query
            const uint32_t tq = lds_address(sT[c & 1][0]), td = lds_address(sT[c & 1][1]);
#pragma unroll
            for (int i = 0; i < IPW; ++i) {
                const int n = wave * IPW + i, r = n * RPI + lane / PPR;
                const long long q = __shfl(idx, r, 64);
                const int piece = ((lane % PPR) ^ (r & 31 & (PPR - 1))) * 16;
                dma16_at(qbase + q * Q.stride_s * 4 + piece, tq + (uint32_t)n * 1024);
                dma16_at(dobase + q * dO.stride_s * 4 + piece, td + (uint32_t)n * 1024);
            }
            if (wave < 2) {
                const float* src = lse_delta + ((long long)bh * 2 + wave) * lse_delta_pitch(S) + idx;
                dma4_at(reinterpret_cast<const char*>(src), lds_address(reinterpret_cast<const char*>(&sLD[c & 1][wave][0])));
            }
        };
        request(0, index_of(0));
        int idx_next = index_of(1);
        const TileReads<D> rd(lane);
        auto next_chunk = [&](int c) {
            VMOBA_WAIT_VMCNT(0);
            __syncthreads();
            if (c + 1 < n_chunks) {
                request(c + 1, idx_next);
                idx_next = index_of(c + 2);
            }
        };
        if (!wave_live) {                                         // no key of this wavefront exists: it only moves rows
            for (int c = 0; c < n_chunks; ++c) next_chunk(c);
        } else
        for (int c = 0; c < n_chunks; ++c) {
            next_chunk(c);
            const char* tQ = sT[c & 1][0] + qh * HALF;
            const char* tdO = sT[c & 1][1] + qh * HALF;
            f32x16_t s = zero16, dp = zero16;
            two_products_over_channels<D>(rd, tQ, tdO, kf, vf, s, dp);
            float oa[DT], qa[DT];
            read_cols<D>(rd, tdO, 0, oa);
            read_cols<D>(rd, tQ, 0, qa);
            const int left = cnt - c * QC - qh * 32 - 4 * hf;      // value 4*i + r is query row 8*i + r of this lane half
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(&sLD[c & 1][0][qh * 32 + 8 * i + 4 * hf]);
                const f32x4_t d4 = *reinterpret_cast<const f32x4_t*>(&sLD[c & 1][1][qh * 32 + 8 * i + 4 * hf]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int v = 4 * i + r;
                    s[v] = exp2_raw(fmaf(s[v], scale_log2, -l4[r]));
                    dp[v] = s[v] * (dp[v] + d4[r]);
                }
            }
            if (left < 32) {                                      // rows past the end of the list
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (8 * (v >> 2) + (v & 3) >= left) { s[v] = 0.f; dp[v] = 0.f; }
            }
            product_over_rows<D>(rd, tdO, oa, s, acc[0]);
            product_over_rows<D>(rd, tQ, qa, dp, acc[1]);
        }
        // the second query half's sums join the first's
        static_assert(2 * 2 * DT * 16 * 64 * 4 <= (int)sizeof(sT), "the sums of two wavefronts fit the row buffers");
        float* red = reinterpret_cast<float*>(&sT[0][0][0]) + kw * (2 * DT * 16 * 64);
        __syncthreads();
        if (qh == 1) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) red[((x * DT + dt) * 16 + v) * 64 + lane] = acc[x][dt][v];
        }
        __syncthreads();
        if (qh == 0) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[x][dt][v] += red[((x * DT + dt) * 16 + v) * 64 + lane];
        }
    }
    if (qh == 0 && live) {
        const long long kout = rows ? rows[krow] : krow;
        float* pv = reinterpret_cast<float*>(dV.ptr + ((long long)b * dV.stride_b + kout * dV.stride_s + (long long)h * dV.stride_h) * 4);
        float* pk = reinterpret_cast<float*>(dK.ptr + ((long long)b * dK.stride_b + kout * dK.stride_s + (long long)h * dK.stride_h) * 4);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t ov = {acc[0][dt][4 * i], acc[0][dt][4 * i + 1], acc[0][dt][4 * i + 2], acc[0][dt][4 * i + 3]};
                const f32x4_t ok = {acc[1][dt][4 * i] * scale, acc[1][dt][4 * i + 1] * scale, acc[1][dt][4 * i + 2] * scale, acc[1][dt][4 * i + 3] * scale};
                *reinterpret_cast<f32x4_t*>(pv + dt * 32 + i * 8 + hf * 4) = ov;
                *reinterpret_cast<f32x4_t*>(pk + dt * 32 + i * 8 + hf * 4) = ok;
            }
    }
}

}  // namespace

void launch_fwd_tiles_f32(int D, dim3 grid, hipStream_t st, const int* run_if, const TensorView& Q, const TensorView& K, const TensorView& V, const int* q_idx,
                          const int4* flat_desc, const int* n_tiles, float* Opart, float* lse_part, int Hh, long long cap,
                          float scale_log2, const int* kv_rows) {
    auto kfn = D == 128 ? attn_fwd_tile_f32_kernel<128> : attn_fwd_tile_f32_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(run_if, Q, K, V, q_idx, flat_desc, n_tiles, Opart, lse_part, Hh, cap, scale_log2, kv_rows);
}

void launch_dq_tiles_f32(int D, dim3 grid, hipStream_t st, const int* run_if, const TensorView& Q, const TensorView& K, const TensorView& V, const TensorView& dO,
                         const float* lse_delta, const int* q_idx, const int4* flat_desc, const int* n_tiles,
                         float* dQpart, int Hh, int S, long long cap, float scale_log2, const int* kv_rows) {
    auto kfn = D == 128 ? attn_bwd_dq_f32_kernel<128> : attn_bwd_dq_f32_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(run_if, Q, K, V, dO, lse_delta, q_idx, flat_desc, n_tiles, dQpart, Hh, S, cap, scale_log2, kv_rows);
}

void launch_dkv_f32(int D, dim3 grid, hipStream_t st, const int* run_if, int parts, const TensorView& Q, const TensorView& K, const TensorView& V, const TensorView& dO,
                    const float* lse_delta, const int* blk_off, const int* blk_ptr, const int* q_idx, const int* kb_start,
                    const int* kb_order, const TensorView& dK, const TensorView& dV, const int* rows, int Hh, int S, int nb, long long cap,
                    float scale_log2, float scale, const int* kv_rows) {
    auto kfn = D == 128 ? attn_bwd_dkv_f32_kernel<128> : attn_bwd_dkv_f32_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(run_if, parts, Q, K, V, dO, lse_delta, blk_off, blk_ptr, q_idx, kb_start, kb_order, dK, dV, rows, Hh, S, nb, cap,
                                    scale_log2, scale, kv_rows);
}
