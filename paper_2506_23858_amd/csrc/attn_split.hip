// Block-sparse attention kernels for float32 tensors on the bfloat16 matrix instruction, for calls large enough to be bound by
// the matrix pipe (the kernels of attn_f32.hip, on the float32 instruction, keep the small ones).
//
// Every float32 operand x is split into three bfloat16 terms, x = h + m + l (each the rounding of what the ones before leave:
// 8 + 8 + 8 mantissa bits, exact to 2^-27 |x| while the last bit stands above bfloat16's smallest number, 2^-133), and a product of two operands is the sum of the six products of terms whose
// orders add up to at most two: h h + (h m + m h) + (h l + l h + m m); what is left out is below 2^-25 |a b|.  Products of terms are
// exact in float32 and summed there, small ones first.  The result is closer to the exact one than the
// float32 instruction's, whose chain of sums is eight times as long per k-step (relative error of a product over 128 / 1024 normal
// values: 1.7e-7 / 5.1e-7 against 2.0e-7 / 5.9e-7), at six 32-cycle instructions for eight of 64 cycles.
//
// Inputs are split once per call, into rows of planes (split_rows_kernel), so that tiles travel from global memory straight to LDS
// and are laid out like the bfloat16 kernels' (RowTile); the soft-max weights and dS are split in registers.
//
// Range.  Terms of an infinity or NaN would not recombine to it, and those of a small number lose its last bits: the split kernel raises
// a flag when it meets a value that is neither 0 nor of a magnitude from 2^-100 up to 2^26, and then these kernels
// leave at once and those of attn_f32.hip, launched behind them, do the work instead.  Weights and dS can be as small as float32
// goes -- a key that no query attends to has only such -- so they are split after a multiplication by 2^16, which makes
// three terms of every normal number exact, and the sums they enter are multiplied by 2^-16 when they are
// written.  With inputs below 2^26 the largest sum, dK' of 2^22 queries, stays below 2^124.
//
// Work decomposition, orientation and operand plumbing as in the bfloat16 kernels (attn_common.h).
//
// Measured on 14 040 tokens x 12 heads x 128 (36 blocks of 390 keys, 785 K kept pairs), float32 instruction -> these: forward
// 1.45 -> 0.80 ms, dQ 2.3 -> 1.26 ms, dK/dV 3.4 -> 1.86 ms, and 0.27 ms for the seven splitting passes (5.5 TB/s); the whole training step
// 7.56 -> 4.8 ms.  Matrix pipe: 60 to 65 % of its rate under load; the rest is a quarter of the last runs' keys (dK/dV),
// the start of a tile with one workgroup per compute unit (dQ), and the soft-max between the products (forward).  Two sums in
// turn for the six products of a k-step instead of one: no faster, spills in the forward kernel, and larger errors in dK and dV.
// Two float16 terms, scaled by a power of two per head, and three products take 3.0 ms for the step, but single rows and channels far below a head's
// largest, and weights far below a key's largest, do not fit five bits of exponent beside it: dV and dK of such a key were wrong by up to 35 %.
#include "attn_common.h"

namespace {

constexpr float LN2 = 0.6931471805599453f;
constexpr float LIFT = 0x1p16f, UNLIFT = 0x1p-16f;                                // of weights and dS, see above
constexpr uint32_t SMALLEST = 27u << 23, TOO_LARGE = 153u << 23;                  // 2^-100 and 2^26 as float bits

// two floats -> their bfloat16 pairs h, m, l (low half = a)
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = pack_bf16x2(a, b);
    const float ra = a - bf16lo_to_f32(h), rb = b - bf16hi_to_f32(h);
    m = pack_bf16x2(ra, rb);
    l = pack_bf16x2(ra - bf16lo_to_f32(m), rb - bf16hi_to_f32(m));
}

// Rows of X (float32, row map[r] of it where a map is given) -> planes h, m, l at plane0 .. plane0 + 2 of row r of dst
// [BH][S][planes][D].  One thread per eight channels.  Bound by HBM: 4 bytes in, 6 out per value.
template <int D>
__global__ __launch_bounds__(256) void split_rows_kernel(TensorView X, const int* __restrict__ map, char* __restrict__ dst, int planes, int plane0, int Hh,
                                                         int S, int* __restrict__ out_of_range) {
    constexpr int PPR = D / 8;
    const int bh = blockIdx.y, b = bh / Hh, h = bh % Hh;
    const int r = blockIdx.x * (256 / PPR) + threadIdx.x / PPR, piece = threadIdx.x % PPR;
    if (r >= S) return;
    const long long src = map ? map[r] : r;
    const f32x4_t* x = reinterpret_cast<const f32x4_t*>(X.ptr + ((long long)b * X.stride_b + src * X.stride_s + (long long)h * X.stride_h) * 4) + piece * 2;
    const f32x4_t v[2] = {x[0], x[1]};
    u32x4_t t[3];
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = v[i >> 1][(i & 1) * 2], c = v[i >> 1][(i & 1) * 2 + 1];
        uint32_t th, tm, tl;
        split2(a, c, th, tm, tl);
        t[0][i] = th; t[1][i] = tm; t[2][i] = tl;
        const uint32_t ua = __float_as_uint(a) & 0x7fffffffu, uc = __float_as_uint(c) & 0x7fffffffu;
        bad |= (ua && ua - SMALLEST >= TOO_LARGE - SMALLEST) || (uc && uc - SMALLEST >= TOO_LARGE - SMALLEST);
    }
    char* d = dst + (((long long)bh * S + r) * planes + plane0) * (D * 2) + piece * 16;
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4_t*>(d + p * D * 2) = t[p];
    if (__ballot(bad) && (threadIdx.x & 63) == 0) atomicOr(out_of_range, 1);
}

// The terms of 16 values per lane in accumulator order, as the B operand of a product over the tile's rows: filled pair by pair.
struct Terms {
    uint32_t t[3][8];
    __device__ __forceinline__ void pair(int j, float a, float b) {
        split2(a, b, t[0][j], t[1][j], t[2][j]);
        asm volatile("" : "+v"(t[0][j]), "+v"(t[1][j]), "+v"(t[2][j]));       // here, not where it is used
    }
    __device__ __forceinline__ void operand(int s, bf16x8_t (&b)[3]) const {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const u32x4_t u = {t[p][4 * s], t[p][4 * s + 1], t[p][4 * s + 2], t[p][4 * s + 3]};
            b[p] = __builtin_bit_cast(bf16x8_t, u);
        }
    }
};
// c += a . b by terms, small products first.  SWAP: in the order of c += b . a, so that a product computed with its operands the other
// way round has the same rounding errors (the weights that dK/dV recomputes then match the LSE they are normalised by).
template <bool SWAP>
__device__ __forceinline__ f32x16_t mfma6(const bf16x8_t (&a)[3], const bf16x8_t (&b)[3], f32x16_t c) {
    constexpr int X = SWAP ? 0 : 2, Y = SWAP ? 0 : 1;
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[X], b[2 - X], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2 - X], b[X], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[Y], b[1 - Y], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1 - Y], b[Y], c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], c, 0, 0, 0);
}

// Tiles of 32 rows x 3 planes in LDS (plane p of a tile HB bytes after plane p - 1) and the requests that fill them.
template <int D>
struct SplitTile : RowTile<D> {
    using TL = RowTile<D>;
    static constexpr int KSTEPS = D / 16, DT = D / 32;
    static constexpr int TILE = 3 * TL::HB;
    static constexpr int REQ = 3 * 32 / TL::RPI;         // requests per tile, shared by four wavefronts
    static constexpr int IPW = REQ / 4;
    static_assert(IPW * 4 == REQ, "equal shares");
    uint32_t rl[TL::NRB], tl[2][TL::NTB];
    __device__ __forceinline__ SplitTile(int lane) {
#pragma unroll
        for (int k = 0; k < TL::NRB; ++k) rl[k] = TL::row_lane(lane, k);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int dt = 0; dt < TL::NTB; ++dt) tl[t][dt] = TL::tr_lane(lane, t, dt);
    }
    __device__ __forceinline__ void rows3(const char* tile, int ks, bf16x8_t (&a)[3]) const {
#pragma unroll
        for (int p = 0; p < 3; ++p) a[p] = TL::rows(tile + p * TL::HB, rl, 0, ks);
    }
    __device__ __forceinline__ void transposed3(const char* tile, int u, bf16x8_t (&a)[3]) const {
#pragma unroll
        for (int p = 0; p < 3; ++p) a[p] = TL::transposed(tile + p * TL::HB, tl, 0, u / DT, u % DT);
    }
    // request i of wavefront `wave` for a tile at LDS address lds: row (of 32) this lane's lanes fetch, and the plane
    __device__ static __forceinline__ int req_row(int wave, int i, int lane) { return (wave * IPW + i) % (32 / TL::RPI) * TL::RPI + lane / TL::PPR; }
    __device__ static __forceinline__ int req_plane(int wave, int i) { return (wave * IPW + i) / (32 / TL::RPI); }
    __device__ static __forceinline__ uint32_t req_lds(int wave, int i) {
        return (uint32_t)(req_plane(wave, i) * TL::HB + (wave * IPW + i) % (32 / TL::RPI) * TL::GP);
    }
    // Vector work of eight value pairs goes between the matrix instructions of a product, PAIRS pairs after every group of six
    // (a wavefront alone on its SIMD would leave the matrix pipe idle for it).
    static constexpr int PAIRS = 8 / KSTEPS;
    static_assert(KSTEPS == 2 * DT, "as many groups in a product over channels as over rows");
    // product over channels: [row rho, column] = tile . f; side(pair) as above
    template <bool SWAP = false, class F>
    __device__ __forceinline__ f32x16_t over_channels(const char* tile, const bf16x8_t (&f)[3][KSTEPS], F&& side) const {
        f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        bf16x8_t a[2][3];
        rows3(tile, 0, a[0]);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            if (ks + 1 < KSTEPS) rows3(tile, ks + 1, a[(ks + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8_t b[3] = {f[0][ks], f[1][ks], f[2][ks]};
            acc = mfma6<SWAP>(a[ks & 1], b, acc);
#pragma unroll
            for (int j = 0; j < PAIRS; ++j) side(ks * PAIRS + j);
            __builtin_amdgcn_sched_barrier(0);
        }
        return acc;
    }
    // product over the tile's rows: acc[dt] += tile^T . w.  With LATE the second half of w's pairs is filled by `side` on the way
    // (side(pair) for pairs 4 .. 7), otherwise w is complete and side runs over all eight pairs of something else.
    template <bool LATE, class F>
    __device__ __forceinline__ void over_rows(const char* tile, const Terms& w, f32x16_t (&acc)[DT], F&& side) const {
        bf16x8_t b[3], a[2][3];
        transposed3(tile, 0, a[0]);
#pragma unroll
        for (int u = 0; u < 2 * DT; ++u) {
            if (u + 1 < 2 * DT) transposed3(tile, u + 1, a[(u + 1) & 1]);
            if (u % DT == 0) w.operand(u / DT, b);
            __builtin_amdgcn_sched_barrier(0);
            acc[u % DT] = mfma6<false>(a[u & 1], b, acc[u % DT]);
            if constexpr (LATE) {
                if (u < DT)
#pragma unroll
                    for (int j = 0; j < 4 / DT; ++j) side(4 + u * (4 / DT) + j);
            } else {
#pragma unroll
                for (int j = 0; j < PAIRS; ++j) side(u * PAIRS + j);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

template <int D>
__device__ __forceinline__ void load_terms(const char* row, int hf, bf16x8_t (&f)[3][D / 16]) {
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) f[p][ks] = *reinterpret_cast<const bf16x8_t*>(row + (p * D + ks * 16 + hf * 8) * 2);
}

// ---------------------------------------------------------------------------------------------
// Forward tile kernel: 4 wavefronts x 32 gathered queries, one key block, 32 keys at a time.  One buffer for K and one for V: the next
// keys are requested as soon as S^T of these is complete, the next values after O^T; two workgroups per compute unit fill
// each other's waits.
template <int D>
__global__ __launch_bounds__(256, 2) void attn_fwd_tile_split_kernel(const char* __restrict__ Q3, const char* __restrict__ KV6, const int* __restrict__ q_idx,
                                                                     const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles,
                                                                     const int* __restrict__ out_of_range, float* __restrict__ Opart,
                                                                     float* __restrict__ lse_part, int S, long long cap, float scale_log2) {
    using ST = SplitTile<D>;
    constexpr int DT = ST::DT, IPW = ST::IPW, RB6 = 12 * D;
    __shared__ __align__(1024) char smem[2 * ST::TILE];
    Tile t;
    if (*out_of_range || !take_tile(flat_desc, n_tiles, t)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long seg = (long long)t.bh * cap;
    const int ent = wave * 32 + l32;
    const int q = q_idx[seg + t.list0 + min(ent, t.count - 1)];   // surplus rows repeat the tile's last query
    const char* kv = KV6 + (long long)t.bh * S * RB6;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t pc16 = ST::request_piece(lane);
    auto request = [&](int c, int tensor) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const uint32_t row = (uint32_t)(t.k0 + min(c * 32 + ST::req_row(wave, i, lane), t.L - 1));
            dma_row16<0>(kv, row, RB6, pc16 + (uint32_t)(tensor * 3 + ST::req_plane(wave, i)) * (2 * D), lds0 + (uint32_t)(tensor * ST::TILE) + ST::req_lds(wave, i));
        }
    };
    request(0, 0);
    request(0, 1);
    bf16x8_t qf[3][ST::KSTEPS];
    load_terms<D>(Q3 + ((long long)t.bh * S + q) * (6 * D), hf, qf);
    const ST st(lane);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16;
    float m_run = -INFINITY, l_run = 0.f;                         // l_run: this lane half's share of the row sum
    const int n_chunks = (t.L + 31) / 32;
    for (int c = 0; c < n_chunks; ++c) {
        VMOBA_WAIT_VMCNT(IPW);                                    // the keys have landed, the values (younger) may be on their way
        __syncthreads();
        f32x16_t s = st.over_channels(smem, qf, [](int) {});
        __syncthreads();                                          // everybody is done with the keys
        request(min(c + 1, n_chunks - 1), 0);                     // (after the last chunk: its own keys again, so that the waits count alike)
        const int left = t.L - c * 32 - hf;                       // value v is key acc_row(v, 0) of this lane half
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] *= scale_log2;          // (a scale of any sign: scaled before the maximum)
        if (left < 32) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (acc_row(v, 0) >= left) s[v] = -INFINITY;
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
        Terms w;
        auto weights = [&](int j) __attribute__((always_inline)) {
            const float p0 = exp2_raw(s[2 * j] - m_run), p1 = exp2_raw(s[2 * j + 1] - m_run);
            l_run += p0 + p1;
            w.pair(j, p0 * LIFT, p1 * LIFT);
        };
#pragma unroll
        for (int j = 0; j < 4; ++j) weights(j);
        VMOBA_WAIT_VMCNT(IPW);                                    // the values have landed
        __syncthreads();
        st.template over_rows<true>(smem + ST::TILE, w, acc, weights);
        __syncthreads();                                          // everybody is done with the values
        request(min(c + 1, n_chunks - 1), 1);
    }
    const float l_tot = swap_halves_sum(l_run);
    if (ent < t.count) {
        const long long pair = seg + t.list0 + ent;
        const float inv = 1.f / l_tot * UNLIFT;
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
    VMOBA_WAIT_VMCNT(0);                                          // no request may reach LDS that belongs to another workgroup by then
}

// ---------------------------------------------------------------------------------------------
// dQ tile kernel: S^T, dP^T, dS^T = P^T (dP^T - delta), dQ^T += K^T dS^T.  The terms of Q and dO take 192 registers: one wavefront per
// SIMD, and a second buffer for the next keys and values.
template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_dq_split_kernel(const char* __restrict__ QD6, const char* __restrict__ KV6,
                                                                   const float* __restrict__ lse_delta, const int* __restrict__ q_idx,
                                                                   const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles,
                                                                   const int* __restrict__ out_of_range, float* __restrict__ dQpart, int S, int pitch,
                                                                   long long cap, float scale_log2) {
    using ST = SplitTile<D>;
    constexpr int DT = ST::DT, IPW = ST::IPW, RB6 = 12 * D;
    __shared__ __align__(1024) char smem[2][2 * ST::TILE];
    Tile t;
    if (*out_of_range || !take_tile(flat_desc, n_tiles, t)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long seg = (long long)t.bh * cap;
    const int ent = wave * 32 + l32;
    const int q = q_idx[seg + t.list0 + min(ent, t.count - 1)];
    const char* kv = KV6 + (long long)t.bh * S * RB6;
    const uint32_t pc16 = ST::request_piece(lane);
    auto request = [&](int c) {
        const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem[c & 1];
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const uint32_t row = (uint32_t)(t.k0 + min(c * 32 + ST::req_row(wave, i, lane), t.L - 1));
            const uint32_t off = pc16 + (uint32_t)ST::req_plane(wave, i) * (2 * D), l = lds + ST::req_lds(wave, i);
            dma_row16<0>(kv, row, RB6, off, l);
            dma_row16<ST::TILE>(kv, row, RB6, off + 6 * D, l);
        }
    };
    request(0);
    bf16x8_t qf[3][ST::KSTEPS], dof[3][ST::KSTEPS];
    load_terms<D>(QD6 + ((long long)t.bh * S + q) * RB6, hf, qf);
    load_terms<D>(QD6 + ((long long)t.bh * S + q) * RB6 + 6 * D, hf, dof);
    const float lse2 = lse_delta[(long long)t.bh * 2 * pitch + q];
    const float ndl = lse_delta[((long long)t.bh * 2 + 1) * pitch + q];
    const ST st(lane);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16;
    const int n_chunks = (t.L + 31) / 32;
    for (int c = 0; c < n_chunks; ++c) {
        VMOBA_WAIT_VMCNT(0);
        __syncthreads();                                          // chunk c has landed; everybody is done with chunk c - 1
        if (c + 1 < n_chunks) request(c + 1);
        const char* sK = smem[c & 1];
        const char* sV = smem[c & 1] + ST::TILE;
        const f32x16_t s = st.over_channels(sK, qf, [](int) {});
        float p[16];
        const f32x16_t dp = st.over_channels(sV, dof, [&](int j) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 2 * j; v < 2 * j + 2; ++v) {
                p[v] = exp2_raw(fmaf(s[v], scale_log2, -lse2)) * LIFT;
                asm volatile("" : "+v"(p[v]));
            }
        });
        const int left = t.L - c * 32 - hf;                       // value v is key acc_row(v, 0) of this lane half
        if (left < 32) {                                          // keys past the block's end: weight 0 (whatever the sign of the scale)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (acc_row(v, 0) >= left) p[v] = 0.f;
        }
        Terms w;
        auto ds_pair = [&](int j) __attribute__((always_inline)) { w.pair(j, p[2 * j] * (dp[2 * j] + ndl), p[2 * j + 1] * (dp[2 * j + 1] + ndl)); };
#pragma unroll
        for (int j = 0; j < 4; ++j) ds_pair(j);
        st.template over_rows<true>(sK, w, acc, ds_pair);
    }
    if (ent < t.count) {
        float* dst = dQpart + (seg + t.list0 + ent) * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t o = {acc[dt][4 * i] * UNLIFT, acc[dt][4 * i + 1] * UNLIFT, acc[dt][4 * i + 2] * UNLIFT, acc[dt][4 * i + 3] * UNLIFT};
                *reinterpret_cast<f32x4_t*>(dst + dt * 32 + i * 8 + hf * 4) = o;
            }
    }
}

// ---------------------------------------------------------------------------------------------
// dK/dV: a workgroup owns 128 keys of one block (32 per wavefront, key = lane % 32) and walks the block's query list 32 queries at a
// time: S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  The LDS holds the six planes of two such chunks.  (Runs of
// 128 keys although a block's last one is rarely full: a second 32-query half per chunk does not fit the LDS.)
template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkv_split_kernel(
    const char* __restrict__ QD6, const char* __restrict__ KV6, const float* __restrict__ lse_delta, const int* __restrict__ blk_off,
    const int* __restrict__ blk_ptr, const int* __restrict__ q_idx, const int* __restrict__ kb_start, const int* __restrict__ kb_order,
    const int* __restrict__ out_of_range, TensorView dK, TensorView dV, const int* __restrict__ rows, int Hh, int S, int pitch, int nb, long long cap,
    float scale_log2, float scale, int BH, int slots, int group) {
    using ST = SplitTile<D>;
    constexpr int DT = ST::DT, IPW = ST::IPW, RB6 = 12 * D;
    __shared__ __align__(1024) char smem[2][2 * ST::TILE];        // [buffer][Q, dO]
    __shared__ float sLD[2][64];                                  // [buffer]: LSE, -delta in accumulator order
    if (*out_of_range) return;
    // groups of one block's runs to the XCDs in turn, heads inside a group number (see attn_bwd_dkv_kernel): 2.51 -> 2.22 ms
    const int n = (int)blockIdx.x >> 3, G = (n / group) * 8 + ((int)blockIdx.x & 7);
    if (G >= BH * (slots / group)) return;
    const int bh = G % BH, run_id = (G / BH) * group + n % group;
    const int b = bh / Hh, h = bh % Hh;
    const int* ks = kb_start + (long long)bh * (nb + 1);
    int lo = 0, hi = nb;
    if (run_id >= ks[nb]) return;
    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (ks[mid] <= run_id) lo = mid; else hi = mid; }
    const int key0 = (run_id - ks[lo]) * 128 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) * 32;     // this wavefront's
    const int j = kb_order[(long long)bh * nb + lo];
    const int k0 = blk_off[j], L = blk_off[j + 1] - k0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int kk = key0 + l32;
    const bool live = kk < L;
    const bool wave_live = key0 < L;                              // any key of this wavefront exists
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
        bf16x8_t kf[3][ST::KSTEPS], vf[3][ST::KSTEPS];
        load_terms<D>(KV6 + ((long long)bh * S + krow) * RB6, hf, kf);
        load_terms<D>(KV6 + ((long long)bh * S + krow) * RB6 + 6 * D, hf, vf);
        const char* qd = QD6 + (long long)bh * S * RB6;
        const char* ldb = reinterpret_cast<const char*>(lse_delta + (long long)bh * 2 * pitch);
        const int* list = q_idx + seg + list0;
        const int n_chunks = (cnt + 31) / 32;
        const uint32_t pc16 = ST::request_piece(lane);
        // lane l % 32 = position p of the accumulator order holds row ld_row; lanes 0..31 LSE, 32..63 -delta
        const int ld_row = ((l32 & 3) << 2) | (((l32 >> 2) & 1) << 1) | (((l32 >> 3) & 1) << 4) | (l32 >> 4);
        auto index_of = [&](int c) { return list[min(c * 32 + l32, cnt - 1)]; };     // lane % 32 = row of the chunk
        auto request = [&](int c, int idx) {                      // rows past the list repeat its last query, with weight 0
            const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem[c & 1];
            const uint32_t ldl = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(char*)&sLD[c & 1][0];
#pragma unroll
            for (int i = 0; i < IPW; ++i) {
                const uint32_t q = (uint32_t)__shfl(idx, ST::req_row(wave, i, lane), 64);
                const uint32_t off = pc16 + (uint32_t)ST::req_plane(wave, i) * (2 * D), l = lds + ST::req_lds(wave, i);
                dma_row16<0>(qd, q, RB6, off, l);
                dma_row16<ST::TILE>(qd, q, RB6, off + 6 * D, l);
            }
            uint32_t lq = (uint32_t)__shfl(idx, ld_row, 64);      // (by every lane: a shuffle reads active lanes only)
            if (c * 32 + ld_row >= cnt) lq = (uint32_t)S;
            if (wave == 0) dma4(ldb, lq * 4 + (hf ? (uint32_t)pitch * 4 : 0u), ldl);
        };
        request(0, index_of(0));
        int idx_next = index_of(1);
        const ST st(lane);
        for (int c = 0; c < n_chunks; ++c) {
            VMOBA_WAIT_VMCNT(0);
            __syncthreads();
            if (c + 1 < n_chunks) {
                request(c + 1, idx_next);
                idx_next = index_of(c + 2);
            }
            if (!wave_live) continue;                             // no key of this wavefront exists: it only moves rows
            const char* tQ = smem[c & 1];
            const char* tdO = smem[c & 1] + ST::TILE;
            const float* ld = &sLD[c & 1][hf * 16];
            const f32x16_t s = st.template over_channels<true>(tQ, kf, [](int) {});
            float p[16];
            Terms pw, dw;
            const f32x16_t dp = st.template over_channels<true>(tdO, vf, [&](int j) __attribute__((always_inline)) {
#pragma unroll
                for (int v = 2 * j; v < 2 * j + 2; ++v) p[v] = exp2_raw(fmaf(s[v], scale_log2, -ld[v])) * LIFT;
                pw.pair(j, p[2 * j], p[2 * j + 1]);
            });
            st.template over_rows<false>(tdO, pw, acc[0], [&](int j) __attribute__((always_inline)) {
                dw.pair(j, p[2 * j] * (dp[2 * j] + ld[32 + 2 * j]), p[2 * j + 1] * (dp[2 * j + 1] + ld[32 + 2 * j + 1]));
            });
            st.template over_rows<false>(tQ, dw, acc[1], [](int) {});
        }
    }
    if (live) {
        const long long kout = rows ? rows[krow] : krow;
        float* pv = reinterpret_cast<float*>(dV.ptr + ((long long)b * dV.stride_b + kout * dV.stride_s + (long long)h * dV.stride_h) * 4);
        float* pk = reinterpret_cast<float*>(dK.ptr + ((long long)b * dK.stride_b + kout * dK.stride_s + (long long)h * dK.stride_h) * 4);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4_t ov, ok;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    ov[r] = acc[0][dt][4 * i + r] * UNLIFT;
                    ok[r] = acc[1][dt][4 * i + r] * UNLIFT * scale;
                }
                *reinterpret_cast<f32x4_t*>(pv + dt * 32 + i * 8 + hf * 4) = ov;
                *reinterpret_cast<f32x4_t*>(pk + dt * 32 + i * 8 + hf * 4) = ok;
            }
    }
}

}  // namespace

void launch_split_rows(int D, int BH, int Hh, int S, hipStream_t st, const TensorView& X, const int* map, char* dst, int planes, int plane0, int* out_of_range) {
    const dim3 grid((unsigned)ceil_div64(S, 256 / (D / 8)), (unsigned)BH);
    auto kfn = D == 128 ? split_rows_kernel<128> : split_rows_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(X, map, dst, planes, plane0, Hh, S, out_of_range);
}

void launch_fwd_tiles_split(int D, dim3 grid, hipStream_t st, const char* Q3, const char* KV6, const int* q_idx, const int4* flat_desc,
                            const int* n_tiles, const int* out_of_range, float* Opart, float* lse_part, int S, long long cap, float scale_log2) {
    auto kfn = D == 128 ? attn_fwd_tile_split_kernel<128> : attn_fwd_tile_split_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(Q3, KV6, q_idx, flat_desc, n_tiles, out_of_range, Opart, lse_part, S, cap, scale_log2);
}

void launch_dq_tiles_split(int D, dim3 grid, hipStream_t st, const char* QD6, const char* KV6, const float* lse_delta, const int* q_idx,
                           const int4* flat_desc, const int* n_tiles, const int* out_of_range, float* dQpart, int S, int pitch, long long cap,
                           float scale_log2) {
    auto kfn = D == 128 ? attn_bwd_dq_split_kernel<128> : attn_bwd_dq_split_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(QD6, KV6, lse_delta, q_idx, flat_desc, n_tiles, out_of_range, dQpart, S, pitch, cap, scale_log2);
}

void launch_dkv_split(int D, dim3 grid, hipStream_t st, const char* QD6, const char* KV6, const float* lse_delta, const int* blk_off, const int* blk_ptr,
                      const int* q_idx, const int* kb_start, const int* kb_order, const int* out_of_range, const TensorView& dK, const TensorView& dV,
                      const int* rows, int Hh, int S, int pitch, int nb, long long cap, float scale_log2, float scale, int BH, int slots, int group) {
    auto kfn = D == 128 ? attn_bwd_dkv_split_kernel<128> : attn_bwd_dkv_split_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(QD6, KV6, lse_delta, blk_off, blk_ptr, q_idx, kb_start, kb_order, out_of_range, dK, dV, rows, Hh, S, pitch, nb,
                                    cap, scale_log2, scale, BH, slots, group);
}
