// Block-sparse attention kernels for float32 tensors on the float16 matrix instruction, for calls large enough to be bound by
// the matrix pipe (the kernels of attn_f32.hip, on the float32 instruction, keep the small ones).
//
// Every float32 operand x, scaled by a power of two, is split into two float16 terms, x = h + l (each the rounding to 11 bits of what is left:
// exact to 2^-23 |x|, and l's sign is a bit of its own, so three values of four are exact), and a product of two operands is the sum of
// three products of terms, h l + l h + h h; what is left out is below 2^-22 |a b|.  Products of terms are exact in float32 and summed there, small
// ones first.  The result is closer to the exact one than the float32 instruction's, whose chain of sums is 16 times as long per
// k-step, and than that of three bfloat16 terms and six products, twice as long: the roundings of the sums are what
// counts (relative error against float64 in profiles/float32_error_against_float64.md), at three 32-cycle instructions for eight of 64 cycles.
//
// Inputs are split once per call, into rows of planes (split_rows_kernel), so that tiles travel from global memory straight to LDS
// and are laid out like the bfloat16 kernels' (RowTile); the soft-max weights and dS are split in registers.
//
// Range.  float16 has 5 bits of exponent, so every tensor of a head is scaled by the power of two that brings its largest magnitude into [2^14, 2^15)
// (split_scan_kernel finds it).  A row whose largest value is 2^-13 of that still has every value down to 2^-24 of
// its own largest exact to 2^-24 of it.  The scan raises a flag where that does not hold -- a row that is not 0 and lies further below the head's largest
// value, an infinity, a NaN, or a head whose largest magnitude is not 0 and outside 2^-100 to 2^26 -- and then these kernels
// leave at once and those of attn_f32.hip, launched behind them, do the work instead.  Soft-max weights enter O and dQ next to a weight near 1
// of the same row, so 2^15 is their scale and their terms are exact to 2^-40.  In dK and dV a key may have only small
// ones -- one that no query attends to -- so there every key has a scale of its own for its weights and one for its dS = P (dP - delta), which are lowered
// when a larger value appears.  In dQ a query's weights have such a scale, and its dS the bound on |dP - delta| that follows from its row of dO.
//
// Work decomposition, orientation and operand plumbing as in the bfloat16 kernels (attn_common.h).
//
// Measured on 14 040 tokens x 12 heads x 128 (36 blocks of 390 keys, 785 K kept pairs), float32 instruction -> three bfloat16 terms and six products -> these:
// forward 1.45 -> 0.81 -> 0.50 ms, dQ 2.3 -> 1.4 -> 0.72 ms, dK/dV 3.4 -> 2.1 -> 1.07 ms, splitting 0 -> 0.27 -> 0.30 ms (5.9 TB/s); the whole
// training step 7.56 -> 4.68 -> 2.98 ms.  Matrix pipe: 50 % of its cycles (forward 52, dQ 50, dK/dV 48); the rest is a workgroup's gathered rows and partial rows
// (dQ, forward: two workgroups per compute unit fill a part of it), the uneven end of the launch (a sixth, dQ and dK/dV) and, in dK/dV, an in-order
// stream of 2.5 vector and 1.2 LDS instructions per matrix instruction on one wavefront per SIMD.
#include "attn_common.h"

namespace {

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));

constexpr float LN2 = 0.6931471805599453f;
constexpr int LIFT = 15;                          // weights are multiplied by 2^LIFT before they are split
constexpr int DQ_LIFT_MOST = 60;                  // of a query's weights in dQ: those of its other blocks count beside them
constexpr int DS_DROP = 38;                       // |dP - delta| at the scales of dO and V is below 2 D 2^15 2^15 <= 2^38
constexpr int LIFT_MOST = 140;                    // of a key's weights in dK and dV: 2^-126 comes to 2^14
constexpr int RING = 4;                            // operands of matrix instructions on their way, see groups()
constexpr int ROW_SPAN = 13;                      // binary orders that the largest values of a head's rows may be apart

// two floats -> their float16 pairs h, l (low half = a)
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& l) {
    const f32x2_t v = {a, b};
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
    f32x2_t r;                                    // what h leaves (the compiler takes two instructions for each)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r.x) : "v"(h), "v"(a));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r.y) : "v"(h), "v"(b));
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2_t));
}

// Largest of the values of the L (8, 16) lanes of a row; every lane receives it.
template <int L>
__device__ __forceinline__ uint32_t row_max(uint32_t x) {
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true));        // lane ^ 1
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xf, 0xf, true));        // lane ^ 2
    x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xf, 0xf, true));       // 7 - lane, of 8
    if constexpr (L == 16) x = max(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x140, 0xf, 0xf, true));   // 15 - lane, of 16
    return x;
}
__device__ __forceinline__ uint2 wave_max_min(uint2 v) {
#pragma unroll
    for (int o = 32; o; o >>= 1) {
        v.x = max(v.x, (uint32_t)__shfl_xor((int)v.x, o, 64));
        v.y = min(v.y, (uint32_t)__shfl_xor((int)v.y, o, 64));
    }
    return v;
}

template <int D>
struct SplitRow {                                                 // eight channels per lane
    static constexpr int PPR = D / 8, ROWS = 256 / PPR;           // lanes per row, rows per step of a workgroup
    f32x4_t v[2];
    __device__ __forceinline__ void load(const SplitTensor& t, int b, int h, long long row, int piece) {
        const f32x4_t* x = reinterpret_cast<const f32x4_t*>(t.X.ptr + ((long long)b * t.X.stride_b + row * t.X.stride_s + (long long)h * t.X.stride_h) * 4) + piece * 2;
        v[0] = x[0]; v[1] = x[1];
    }
};

// Largest magnitude of a tensor's head and the smallest of its rows' largest (rows of zeros aside), as float bits, for chunk blockIdx.x of its
// rows: partial[tensor][head][chunk].  An infinity or NaN counts as the largest.  Bound by HBM.
template <int D>
__global__ __launch_bounds__(256) void split_scan_kernel(SplitTensors in, uint2* __restrict__ partial, int Hh, int S) {
    using R = SplitRow<D>;
    __shared__ uint2 sW[4];
    const int bh = blockIdx.y, b = bh / Hh, h = bh % Hh;
    const SplitTensor& t = in.t[blockIdx.z];
    const int per = (S + gridDim.x - 1) / gridDim.x, r0 = blockIdx.x * per, r1 = min(S, r0 + per);
    const int piece = threadIdx.x % R::PPR;
    uint2 mm = {0u, 0xffffffffu};
    for (int r = r0 + (int)threadIdx.x / R::PPR; r < r1; r += 4 * R::ROWS) {
        R x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i].load(t, b, h, min(r + i * R::ROWS, r1 - 1), piece);      // (the last row again: no harm)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t m = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c) m = max(m, __float_as_uint(x[i].v[c >> 2][c & 3]) & 0x7fffffffu);
            m = row_max<R::PPR>(m);
            mm.x = max(mm.x, m);
            if (m) mm.y = min(mm.y, m);
        }
    }
    mm = wave_max_min(mm);
    if ((threadIdx.x & 63) == 0) sW[threadIdx.x >> 6] = mm;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) { mm.x = max(mm.x, sW[w].x); mm.y = min(mm.y, sW[w].y); }
        partial[((long long)blockIdx.z * gridDim.y + bh) * gridDim.x + blockIdx.x] = mm;
    }
}

// Rows of a tensor (float32, row map[r] of it where a map is given) -> planes h, l of row r at its place, scaled by 2^power;
// power[head][tensor] is written beside.  One thread per eight channels of four rows.  Bound by HBM: 4 bytes in, 4 out per value.
template <int D>
__global__ __launch_bounds__(256) void split_rows_kernel(SplitTensors in, const uint2* __restrict__ partial, int chunks, int* __restrict__ power, int Hh, int S,
                                                         int* __restrict__ out_of_range) {
    using R = SplitRow<D>;
    const int bh = blockIdx.y, b = bh / Hh, h = bh % Hh, lane = threadIdx.x & 63;
    const SplitTensor& t = in.t[blockIdx.z];
    const int r0 = blockIdx.x * (4 * R::ROWS) + threadIdx.x / R::PPR, piece = threadIdx.x % R::PPR;
    R x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = min(r0 + i * R::ROWS, S - 1);
        x[i].load(t, b, h, t.map ? t.map[r] : r, piece);
    }
    uint2 mm = {0u, 0xffffffffu};
    if (lane < chunks) mm = partial[((long long)blockIdx.z * gridDim.y + bh) * chunks + lane];
    mm = wave_max_min(mm);
    const int e = (int)(mm.x >> 23), e_min = (int)(min(mm.x, mm.y) >> 23);
    const bool bad = mm.x && (e < 127 - 100 || e >= 127 + 26 || e - e_min > ROW_SPAN);
    const int p = mm.x && !bad ? 127 + 14 - e : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        power[bh * 4 + blockIdx.z] = p;
        if (bad) *out_of_range = 1;
    }
    const float up = __uint_as_float((uint32_t)(127 + p) << 23);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = r0 + i * R::ROWS;
        if (r >= S) break;
        u32x4_t th, tl;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t a, c;
            split2(x[i].v[j >> 1][(j & 1) * 2] * up, x[i].v[j >> 1][(j & 1) * 2 + 1] * up, a, c);
            th[j] = a; tl[j] = c;
        }
        char* d = t.dst + ((long long)bh * S + r) * t.pitch + piece * 16;
        *reinterpret_cast<u32x4_t*>(d) = th;
        *reinterpret_cast<u32x4_t*>(d + D * 2) = tl;
    }
}

// The terms of 16 values per lane in accumulator order, as the B operand of a product over the tile's rows: filled pair by pair.
struct Terms {
    uint32_t t[2][8];
    __device__ __forceinline__ void pair(int j, float a, float b) {
        split2(a, b, t[0][j], t[1][j]);
        asm volatile("" : "+v"(t[0][j]), "+v"(t[1][j]));                      // here, not where it is used
    }
    __device__ __forceinline__ void operand(int s, f16x8_t (&b)[2]) const {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const u32x4_t u = {t[p][4 * s], t[p][4 * s + 1], t[p][4 * s + 2], t[p][4 * s + 3]};
            b[p] = __builtin_bit_cast(f16x8_t, u);
        }
    }
};
// Matrix instruction M (0 .. 2) of c += a . b by terms, small products first.  SWAP: in the order of c += b . a, so that a product computed with its
// operands the other way round has the same rounding errors (the weights that dK/dV recomputes then match the LSE they are normalised by).
template <bool SWAP, int M>
__device__ __forceinline__ void mfma_part(const f16x8_t (&a)[2], const f16x8_t (&b)[2], f32x16_t& c) {
    constexpr int I = M == 2 ? 0 : SWAP ? M : 1 - M, J = M == 2 ? 0 : 1 - I;
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[I], b[J], c, 0, 0, 0);
}

// A matrix instruction whose second operand, a fragment that the wavefront keeps for good, lies in accumulator registers: the compiler keeps such fragments there too, once the others
// are full, but copies them before every use (113 copies beside 96 matrix instructions).  ZERO: the first of a sum.  The compiler does not see that the result takes
// its time: sum_ready stands before the first vector instruction that reads it.
template <bool ZERO>
__device__ __forceinline__ void mfma_frag(f32x16_t& d, f16x8_t a, f16x8_t frag) {
    if constexpr (ZERO) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(frag));
    else asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(frag));
}
__device__ __forceinline__ void sum_ready(f32x16_t& d) { asm volatile("s_nop 11" : "+v"(d)); }

// N groups of three matrix instructions; fetch(g, a) asks for the operands of group g, AHEAD groups before mul(g, m, a) issues its instruction m, and
// side(g, m) is what to do behind that: a wavefront issues in order, so what stands between two matrix instructions is hidden behind the first as long as it
// takes no more than its 32 cycles, and what stands behind the second waits for it.  The fetches run past the end: those of groups
// N .. N + AHEAD - 1 are the next call's, whose ring `a` goes on (AHEAD + 1 divides N).
constexpr int AHEAD = RING - 1;
template <int N, class Fetch, class Mul, class Side>
__device__ __forceinline__ void groups(f16x8_t (&a)[RING][2], Fetch&& fetch, Mul&& mul, Side&& side) {
    static_assert(N % RING == 0, "the ring goes on");
    static_for<N>([&](auto g) __attribute__((always_inline)) {
        static_for<3>([&](auto m) __attribute__((always_inline)) {
            mul(g, m, a[g % RING]);
            if constexpr (m == 0) fetch(std::integral_constant<int, g + AHEAD>{}, a[(g + AHEAD) % RING]);
            side(g, m);
            __builtin_amdgcn_sched_barrier(0);
        });
    });
}

// Tiles of 32 rows x 2 planes in LDS (plane l of a tile HB bytes after plane h) and the requests that fill them.
template <int D>
struct SplitTile : RowTile<D> {
    using TL = RowTile<D>;
    static constexpr int KSTEPS = D / 16, DT = D / 32;
    static constexpr int TILE = 2 * TL::HB;
    static constexpr int REQ = 2 * 32 / TL::RPI;         // requests per tile, shared by four wavefronts
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
    __device__ __forceinline__ void rows2(const char* tile, int ks, f16x8_t (&a)[2]) const {
#pragma unroll
        for (int p = 0; p < 2; ++p) a[p] = __builtin_bit_cast(f16x8_t, TL::rows(tile + p * TL::HB, rl, 0, ks));
    }
    __device__ __forceinline__ void transposed2(const char* tile, int u, f16x8_t (&a)[2]) const {
#pragma unroll
        for (int p = 0; p < 2; ++p) a[p] = __builtin_bit_cast(f16x8_t, TL::transposed(tile + p * TL::HB, tl, 0, u / DT, u % DT));
    }
    // request i of wavefront `wave` for a tile at LDS address lds: row (of 32) this lane's lanes fetch, and the plane
    __device__ static __forceinline__ int req_row(int wave, int i, int lane) { return (wave * IPW + i) % (32 / TL::RPI) * TL::RPI + lane / TL::PPR; }
    __device__ static __forceinline__ int req_plane(int wave, int i) { return (wave * IPW + i) / (32 / TL::RPI); }
    __device__ static __forceinline__ uint32_t req_lds(int wave, int i) {
        return (uint32_t)(req_plane(wave, i) * TL::HB + (wave * IPW + i) % (32 / TL::RPI) * TL::GP);
    }
    // Vector work of eight value pairs goes between the matrix instructions of a product, PAIRS pairs after every group of three
    // (a wavefront alone on its SIMD would leave the matrix pipe idle for it).
    static constexpr int PAIRS = 8 / KSTEPS;
    static_assert(KSTEPS == 2 * DT, "as many groups in a product over channels as over rows");
    // product over channels: [row rho, column] = acc + tile . f; side(pair) as above
    template <class F>
    __device__ __forceinline__ f32x16_t over_channels(const char* tile, const f16x8_t (&f)[2][KSTEPS], f32x16_t acc, F&& side) const {
        f16x8_t a[2][2];
        rows2(tile, 0, a[0]);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            if (ks + 1 < KSTEPS) rows2(tile, ks + 1, a[(ks + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            const f16x8_t b[2] = {f[0][ks], f[1][ks]};
            mfma_part<false, 0>(a[ks & 1], b, acc);
            mfma_part<false, 1>(a[ks & 1], b, acc);
            mfma_part<false, 2>(a[ks & 1], b, acc);
#pragma unroll
            for (int j = 0; j < PAIRS; ++j) side(ks * PAIRS + j);
            __builtin_amdgcn_sched_barrier(0);
        }
        return acc;
    }
    // product over the tile's rows: acc[dt] += tile^T . w, of which side(pair) fills pairs 4 .. 7 on the way
    template <class F>
    __device__ __forceinline__ void over_rows(const char* tile, const Terms& w, f32x16_t (&acc)[DT], F&& side) const {
        f16x8_t b[2], a[2][2];
        transposed2(tile, 0, a[0]);
#pragma unroll
        for (int u = 0; u < 2 * DT; ++u) {
            if (u + 1 < 2 * DT) transposed2(tile, u + 1, a[(u + 1) & 1]);
            if (u % DT == 0) w.operand(u / DT, b);
            __builtin_amdgcn_sched_barrier(0);
            mfma_part<false, 0>(a[u & 1], b, acc[u % DT]);
            mfma_part<false, 1>(a[u & 1], b, acc[u % DT]);
            mfma_part<false, 2>(a[u & 1], b, acc[u % DT]);
            if (u < DT)
#pragma unroll
                for (int j = 0; j < 4 / DT; ++j) side(4 + u * (4 / DT) + j);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

template <int D>
__device__ __forceinline__ void load_terms(const char* row, int hf, f16x8_t (&f)[2][D / 16]) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) f[p][ks] = *reinterpret_cast<const f16x8_t*>(row + (p * D + ks * 16 + hf * 8) * 2);
}

// ---------------------------------------------------------------------------------------------
// Forward tile kernel: 4 wavefronts x 32 gathered queries, one key block, 32 keys at a time.  Two buffers of keys and values, requested one
// chunk ahead, one barrier per chunk; two workgroups per compute unit fill each other's waits.
template <int D>
__global__ __launch_bounds__(256, 2) void attn_fwd_tile_split_kernel(const char* __restrict__ Q2, const char* __restrict__ KV4, const int4* __restrict__ power,
                                                                     const int* __restrict__ q_idx, const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles,
                                                                     const int* __restrict__ out_of_range, float* __restrict__ Opart,
                                                                     float* __restrict__ lse_part, int S, long long cap, float scale_log2) {
    using ST = SplitTile<D>;
    constexpr int DT = ST::DT, IPW = ST::IPW, RB4 = 8 * D;
    __shared__ __align__(1024) char smem[2][2 * ST::TILE];
    Tile t;
    if (*out_of_range || !take_tile(flat_desc, n_tiles, t)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long seg = (long long)t.bh * cap;
    const int ent = wave * 32 + l32;
    const int q = q_idx[seg + t.list0 + min(ent, t.count - 1)];   // surplus rows repeat the tile's last query
    const char* kv = KV4 + (long long)t.bh * S * RB4;
    const int4 pw = power[t.bh];                                  // of Q, K, V
    const float sl = ldexpf(scale_log2, -(pw.x + pw.y));
    const uint32_t pc16 = ST::request_piece(lane);
    auto request = [&](int c) {
        const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem[c & 1];
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const uint32_t row = (uint32_t)(t.k0 + min(c * 32 + ST::req_row(wave, i, lane), t.L - 1));
            const uint32_t off = pc16 + (uint32_t)ST::req_plane(wave, i) * (2 * D), l = lds + ST::req_lds(wave, i);
            dma_row16<0>(kv, row, RB4, off, l);
            dma_row16<ST::TILE>(kv, row, RB4, off + 4 * D, l);
        }
    };
    request(0);
    f16x8_t qf[2][ST::KSTEPS];
    load_terms<D>(Q2 + ((long long)t.bh * S + q) * (4 * D), hf, qf);
    const ST st(lane);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16;
    float m_run = -INFINITY, l_run = 0.f;                         // l_run: this lane half's share of the row sum
    const int n_chunks = (t.L + 31) / 32;
    for (int c = 0; c < n_chunks; ++c) {
        VMOBA_WAIT_VMCNT(0);
        __syncthreads();                                          // chunk c has landed; everybody is done with chunk c - 1
        if (c + 1 < n_chunks) request(c + 1);
        const char* sK = smem[c & 1];
        f32x16_t s = st.over_channels(sK, qf, zero16, [](int) {});
        const int left = t.L - c * 32 - hf;                       // value v is key acc_row(v, 0) of this lane half
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] *= sl;                  // (a scale of any sign: scaled before the maximum)
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
            w.pair(j, p0 * (float)(1 << LIFT), p1 * (float)(1 << LIFT));
        };
#pragma unroll
        for (int j = 0; j < 4; ++j) weights(j);
        st.over_rows(sK + ST::TILE, w, acc, weights);
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
                f32x4_t o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = ldexpf(acc[dt][4 * i + r] * inv, -(LIFT + pw.z));
                *reinterpret_cast<f32x4_t*>(dst + dt * 32 + i * 8 + hf * 4) = o;
            }
        if (hf == 0) lse_part[pair] = (m_run + log2f(l_tot)) * LN2;
    }
}

// ---------------------------------------------------------------------------------------------
// dQ tile kernel: S^T, dP^T, dS^T = P^T (dP^T - delta), dQ^T += K^T dS^T.  Two buffers of keys and values, requested one chunk ahead, one barrier per
// chunk.  The terms of Q and dO and the sums take 192 of the 256 registers that two wavefronts per SIMD leave each; six addresses do not fit.  One wavefront
// per SIMD, with dS between the instructions of the next S and three buffers, is slower (0.90 against 0.73 ms): nothing fills the gathers of a tile's start.
template <int D>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_split_kernel(const char* __restrict__ QD4, const char* __restrict__ KV4, const int4* __restrict__ power,
                                                                   const float* __restrict__ lse_delta, const int* __restrict__ q_idx,
                                                                   const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles,
                                                                   const int* __restrict__ out_of_range, float* __restrict__ dQpart, int S, int pitch,
                                                                   long long cap, float scale_log2) {
    using ST = SplitTile<D>;
    constexpr int DT = ST::DT, IPW = ST::IPW, RB4 = 8 * D;
    __shared__ __align__(1024) char smem[2][2 * ST::TILE];
    Tile t;
    if (*out_of_range || !take_tile(flat_desc, n_tiles, t)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const long long seg = (long long)t.bh * cap;
    const int ent = wave * 32 + l32;
    const int q = q_idx[seg + t.list0 + min(ent, t.count - 1)];
    const char* kv = KV4 + (long long)t.bh * S * RB4;
    const uint32_t pc16 = ST::request_piece(lane);
    auto request = [&](int c) {
        const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem[c & 1];
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            const uint32_t row = (uint32_t)(t.k0 + min(c * 32 + ST::req_row(wave, i, lane), t.L - 1));
            const uint32_t off = pc16 + (uint32_t)ST::req_plane(wave, i) * (2 * D), l = lds + ST::req_lds(wave, i);
            dma_row16<0>(kv, row, RB4, off, l);
            dma_row16<ST::TILE>(kv, row, RB4, off + 4 * D, l);
        }
    };
    request(0);
    f16x8_t qf[2][ST::KSTEPS], dof[2][ST::KSTEPS];
    load_terms<D>(QD4 + ((long long)t.bh * S + q) * RB4, hf, qf);
    load_terms<D>(QD4 + ((long long)t.bh * S + q) * RB4 + 4 * D, hf, dof);
    const float lse2 = lse_delta[(long long)t.bh * 2 * pitch + q];
    const int4 pw = power[t.bh];                                  // of Q, dO, K, V
    const float ndl = ldexpf(lse_delta[((long long)t.bh * 2 + 1) * pitch + q], pw.y + pw.w);
    const float sl = ldexpf(scale_log2, -(pw.x + pw.z));
    const ST st(lane);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16;
    // This query's weights are multiplied by 2^lift, and for dS by 2^-drop: below DS_DROP by what the largest value of its row of dO lacks.
    int lift = DQ_LIFT_MOST;
    f16x8_t row = {};
#pragma unroll
    for (int ks = 0; ks < ST::KSTEPS; ++ks) row = __builtin_elementwise_max(row, __builtin_elementwise_abs(dof[0][ks]));
    float row_most = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) row_most = fmaxf(row_most, (float)row[i]);
    row_most = swap_halves_max(row_most);
    const int drop = DS_DROP - 127 - 14 + max((int)(__float_as_uint(row_most) >> 23), 127 - 24);
    const float largest = ldexpf(1.f, LIFT - drop);
    const int n_chunks = (t.L + 31) / 32;
    for (int c = 0; c < n_chunks; ++c) {
        VMOBA_WAIT_VMCNT(0);
        __syncthreads();                                          // chunk c has landed; everybody is done with chunk c - 1
        if (c + 1 < n_chunks) request(c + 1);
        const char* sK = smem[c & 1];
        const char* sV = smem[c & 1] + ST::TILE;
        f32x16_t s = st.over_channels(sK, qf, zero16, [](int) {});
        float most = 0.f;
        const f32x16_t dp = st.over_channels(sV, dof, zero16, [&](int j) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 2 * j; v < 2 * j + 2; ++v) {
                s[v] = ldexpf(exp2_raw(fmaf(s[v], sl, -lse2)), lift - drop);
                most = fmaxf(most, s[v]);
            }
        });
        const int left = t.L - c * 32 - hf;                       // value v is key acc_row(v, 0) of this lane half
        if (left < 32) {                                          // keys past the block's end: weight 0 (whatever the sign of the scale)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (acc_row(v, 0) >= left) s[v] = 0.f;
        }
        if (__builtin_amdgcn_ballot_w64(most > largest)) {        // too large a weight for the query's scale: it becomes about 2^11
            most = swap_halves_max(most);
            const int by = most > largest ? 127 + 11 - drop - (int)(__float_as_uint(most) >> 23) : 0;
            lift += by;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = ldexpf(s[v], by);
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[d][v] = ldexpf(acc[d][v], by);
        }
        Terms w;
        auto ds_pair = [&](int j) __attribute__((always_inline)) { w.pair(j, s[2 * j] * (dp[2 * j] + ndl), s[2 * j + 1] * (dp[2 * j + 1] + ndl)); };
#pragma unroll
        for (int j = 0; j < 4; ++j) ds_pair(j);
        st.over_rows(sK, w, acc, ds_pair);
    }
    if (ent < t.count) {
        float* dst = dQpart + (seg + t.list0 + ent) * D;
        const int down = -(lift - drop + pw.y + pw.w + pw.z);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4_t o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = ldexpf(acc[dt][4 * i + r], down);
                *reinterpret_cast<f32x4_t*>(dst + dt * 32 + i * 8 + hf * 4) = o;
            }
    }
}

// ---------------------------------------------------------------------------------------------
// dK/dV: a workgroup owns a run of 128 keys of one block (32 per wavefront, key = lane % 32) and walks the block's query list 32 queries at a
// time: S = Q K^T, dP = dO V^T (with the weights), dV^T += dO^T P (with dS), dK^T += Q^T dS.  One wavefront per SIMD, three buffers, one barrier, as in dQ.
// HALVES: a run of at most 64 keys -- a block's last one -- goes over two such chunks at a time: wavefronts 2 and 3 have the keys of 0 and 1 and every
// second chunk, and their sums are added at the end (two buffers of two chunks: the operands of a step's first groups are not
// fetched ahead of its barrier).  Such a block of few keys takes a large share of the weights of most queries, and its sums are the longest: a step's share is summed by
// itself and added once (two roundings of a long sum per step and product instead of six).
template <int D>
struct DkvSmem {
    using ST = SplitTile<D>;
    static constexpr int CHUNK = 2 * ST::TILE;                    // Q, dO
    __align__(1024) char rows[4 * CHUNK];
    float ld[4][64];                                              // LSE, -delta in accumulator order
};
struct DkvRun { int bh, b, h, j, k0, L, list0, cnt, first; };     // first: first key of the run inside the block
template <int D, bool HALVES>
__device__ __forceinline__ void dkv_run(DkvSmem<D>& sm, const DkvRun& run, const char* __restrict__ QD4, const char* __restrict__ KV4, const int4 pw,
                                        const float* __restrict__ lse_delta, const int* __restrict__ list, const TensorView& dK, const TensorView& dV,
                                        const int* __restrict__ rows, int S, int pitch, float scale_log2, float scale) {
    using ST = SplitTile<D>;
    constexpr int DT = ST::DT, IPW = ST::IPW, RB4 = 8 * D, G = ST::KSTEPS, PAIRS = ST::PAIRS, CHUNK = DkvSmem<D>::CHUNK;
    constexpr int SUB = HALVES ? 2 : 1, NBUF = HALVES ? 2 : 3;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const int sub = HALVES ? wave >> 1 : 0;
    const int key0 = run.first + (HALVES ? wave & 1 : wave) * 32, kk = key0 + l32;
    const int L = run.L, cnt = run.cnt;
    const bool wave_live = key0 < L;                              // any key of this wavefront exists
    const int krow = run.k0 + min(kk, L - 1);
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int lift = LIFT_MOST, fall = 0;                               // this key's weights are multiplied by 2^lift, its dS by 2^(lift - fall)
    f32x16_t acc[2][DT];                                          // dV^T, dK^T
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc[x][dt] = zero16;
    if (cnt > 0) {                                                // uniform over the workgroup
        f16x8_t kf[2][G], vf[2][G];
        load_terms<D>(KV4 + ((long long)run.bh * S + krow) * RB4, hf, kf);
        load_terms<D>(KV4 + ((long long)run.bh * S + krow) * RB4 + 4 * D, hf, vf);
        const char* qd = QD4 + (long long)run.bh * S * RB4;
        const char* ldb = reinterpret_cast<const char*>(lse_delta + (long long)run.bh * 2 * pitch);
        const int n_steps = (cnt + 32 * SUB - 1) / (32 * SUB);
        const uint32_t pc16 = ST::request_piece(lane);
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)sm.rows;
        const uint32_t ld0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(char*)&sm.ld[0][0];
        // lane l % 32 = position p of the accumulator order holds row ld_row; lanes 0..31 LSE, 32..63 -delta
        const int ld_row = ((l32 & 3) << 2) | (((l32 >> 2) & 1) << 1) | (((l32 >> 3) & 1) << 4) | (l32 >> 4);
        auto index_of = [&](int c) { return list[min(c * (32 * SUB) + (HALVES ? lane : l32), cnt - 1)]; };     // one lane per row of a step
        // Row numbers of a step's requests (looked up all at once: a shuffle's answer takes as long as an LDS read), then the requests.
        constexpr int NREQ = SUB * IPW;
        static_assert(NREQ + 2 <= G || HALVES, "one request per group");
        uint32_t qn[NREQ], lq[SUB];
        auto look_up = [&](int c, int idx) __attribute__((always_inline)) {             // rows past the list repeat its last query, with weight 0
#pragma unroll
            for (int i = 0; i < NREQ; ++i) qn[i] = (uint32_t)__shfl(idx, i / IPW * 32 + ST::req_row(wave, i % IPW, lane), 64);
#pragma unroll
            for (int x = 0; x < SUB; ++x) {
                lq[x] = (uint32_t)__shfl(idx, x * 32 + ld_row, 64);
                if ((c * SUB + x) * 32 + ld_row >= cnt) lq[x] = (uint32_t)S;
            }
        };
        auto request = [&](int slot, int i) __attribute__((always_inline)) {            // (slot: the buffer's first chunk)
            const int x = i / IPW, ii = i % IPW;
            const uint32_t off = pc16 + (uint32_t)ST::req_plane(wave, ii) * (2 * D), l = lds0 + (uint32_t)(slot + x) * CHUNK + ST::req_lds(wave, ii);
            dma_row16<0>(qd, qn[i], RB4, off, l);
            dma_row16<ST::TILE>(qd, qn[i], RB4, off + 4 * D, l);
            if (ii == IPW - 1 && wave == x) dma4(ldb, lq[x] * 4 + (hf ? (uint32_t)pitch * 4 : 0u), ld0 + (uint32_t)(slot + x) * 256);
        };
        int idx = index_of(0);
        look_up(0, idx);
#pragma unroll
        for (int i = 0; i < NREQ; ++i) request(0, i);
        if constexpr (!HALVES) {
            look_up(1, index_of(1));
#pragma unroll
            for (int i = 0; i < NREQ; ++i) request(1, i);
        }
        idx = index_of(NBUF - 1);
        const ST st(lane);
        const float sl = ldexpf(scale_log2, -(pw.x + pw.z));
        constexpr float LARGEST = (float)(1 << LIFT);
        float down = 1.f;                                         // 2^-fall
        f16x8_t a[RING][2];
        f32x16_t s, dp, part[2];                                  // part: HALVES, of a channel tile and the one before
        float p[16];
        Terms pt, dt;
        constexpr int EARLY = HALVES ? 8 : 4;                     // pairs that are split before the product that needs them
        int buf = 0;
        for (int c = 0; c < n_steps; ++c) {
            const int next = buf == NBUF - 1 ? 0 : buf + 1, after = NBUF == 2 ? next : next == 2 ? 0 : next + 1;      // `after` takes what is requested now
            VMOBA_WAIT_VMCNT(0);
            __syncthreads();                                      // this step's rows (HALVES; else the next step's too) have landed; everybody is done with step c - 1
            look_up(c + NBUF - 1, idx);
            if (!wave_live || HALVES) {
#pragma unroll
                for (int i = 0; i < NREQ; ++i) request(after * SUB, i);
                if (!wave_live) {                                 // no key of this wavefront exists: it only moves rows
                    idx = index_of(c + NBUF);
                    buf = next;
                    continue;
                }
            }
            const char* tQ = sm.rows + (buf * SUB + sub) * CHUNK;
            const char* tdO = tQ + ST::TILE;
            const char* tQn = sm.rows + next * CHUNK;
            f32x4_t lse[4], ndl[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                lse[i] = *reinterpret_cast<const f32x4_t*>(&sm.ld[buf * SUB + sub][hf * 16 + 4 * i]);
                ndl[i] = *reinterpret_cast<const f32x4_t*>(&sm.ld[buf * SUB + sub][32 + hf * 16 + 4 * i]);
            }
            float most = 0.f, most_ds = 0.f;
            if (HALVES || c == 0) static_for<AHEAD>([&](auto i) { st.rows2(tQ, i, a[i]); });
            groups<4 * G>(a,
                [&](auto g, f16x8_t (&x)[2]) __attribute__((always_inline)) {
                    if constexpr (g < G) st.rows2(tQ, g, x);
                    else if constexpr (g < 2 * G) st.rows2(tdO, g - G, x);
                    else if constexpr (g < 4 * G) st.transposed2(g < 3 * G ? tdO : tQ, HALVES ? g % 2 * DT + g % G / 2 : g % G, x);
                    else if constexpr (!HALVES) st.rows2(tQn, g - 4 * G, x);
                },
                [&](auto g, auto m, const f16x8_t (&x)[2]) __attribute__((always_inline)) {
                    if constexpr (g < G) {
                        mfma_frag<g == 0 && m == 0>(s, x[m == 1 ? 1 : 0], kf[m == 0 ? 1 : 0][g]);
                    } else if constexpr (g < 2 * G) {
                        mfma_frag<false>(dp, x[m == 1 ? 1 : 0], vf[m == 0 ? 1 : 0][g - G]);
                        if constexpr (g == G && m == 0) sum_ready(s);
                    } else {
                        constexpr int x4 = g < 3 * G ? 0 : 1, u = g % G;
                        f16x8_t b[2];
                        (x4 ? dt : pt).operand(HALVES ? u % 2 : u / DT, b);
                        if constexpr (HALVES) {
                            if constexpr (u % 2 == 0 && m == 0) part[u / 2 % 2] = zero16;
                            mfma_part<false, m>(x, b, part[u / 2 % 2]);
                        } else mfma_part<false, m>(x, b, acc[x4][u % DT]);
                        if constexpr (g == 2 * G && m == 0) sum_ready(dp);
                    }
                },
                [&](auto g, auto m) __attribute__((always_inline)) {
                    if constexpr (g < G) {
                        if constexpr (m == 1 && !HALVES && g >= 2 && g - 2 < NREQ) request(after, g - 2);
                        if constexpr (m == 0 && g >= DT) {
#pragma unroll
                            for (int v = 4 * PAIRS * (g - DT); v < 4 * PAIRS * (g - DT + 1); ++v) dp[v] = ldexpf(ndl[v >> 2][v & 3], pw.y + pw.w);
                        }
                        if constexpr (g == G - 1 && m == 2) idx = index_of(c + NBUF);
                    } else if constexpr (g < 2 * G) {
                        static_for<PAIRS>([&](auto i) __attribute__((always_inline)) {
                            constexpr int j = PAIRS * (g - G) + i;
                            if constexpr (m == 0) {
                                p[2 * j] = exp2_raw(fmaf(s[2 * j], sl, -lse[j >> 1][2 * j & 3]));
                                p[2 * j + 1] = exp2_raw(fmaf(s[2 * j + 1], sl, -lse[j >> 1][(2 * j & 3) + 1]));
                            } else if constexpr (m == 1) {
                                p[2 * j] = ldexpf(p[2 * j], lift);
                                p[2 * j + 1] = ldexpf(p[2 * j + 1], lift);
                                most = fmaxf(most, fmaxf(p[2 * j], p[2 * j + 1]));
                            } else if constexpr (j < EARLY) {
                                pt.pair(j, p[2 * j], p[2 * j + 1]);
                            }
                            asm volatile("" : "+v"(p[2 * j]), "+v"(p[2 * j + 1]));
                        });
                        if constexpr (g == 2 * G - 1 && m == 2) {
                            if (__builtin_amdgcn_ballot_w64(most > LARGEST)) {        // a key's largest weight so far is too large for its scale: it becomes about 2^11
                                float r[16];                      // (computed again: at the old scale they may not be finite)
                                most = 0.f;
#pragma unroll
                                for (int v = 0; v < 16; ++v) { r[v] = exp2_raw(fmaf(s[v], sl, -lse[v >> 2][v & 3])); most = fmaxf(most, r[v]); }
                                most = swap_halves_max(most);
                                const int by = ldexpf(most, lift) > LARGEST ? 127 + 11 - (int)(__float_as_uint(most) >> 23) - lift : 0;
                                lift += by;
#pragma unroll
                                for (int v = 0; v < 16; ++v) p[v] = ldexpf(r[v], lift);
#pragma unroll
                                for (int j = 0; j < EARLY; ++j) pt.pair(j, p[2 * j], p[2 * j + 1]);
#pragma unroll
                                for (int x = 0; x < 2; ++x)
#pragma unroll
                                    for (int d = 0; d < DT; ++d)
#pragma unroll
                                        for (int v = 0; v < 16; ++v) acc[x][d][v] = ldexpf(acc[x][d][v], by);
                            }
                        }
                    } else if constexpr (g < 3 * G + DT) {        // the second halves of the terms on the way, in the first half of the groups that need them
                        static_for<PAIRS>([&](auto i) __attribute__((always_inline)) {
                            constexpr int j = PAIRS * (g % G) + i;
                            if constexpr (g >= 3 * G) {
                                if constexpr (m == 0 && !HALVES) dt.pair(4 + j, p[8 + 2 * j], p[8 + 2 * j + 1]);
                            } else {
                                if constexpr (m == 0) {
                                    p[2 * j] *= down * dp[2 * j];
                                    p[2 * j + 1] *= down * dp[2 * j + 1];
                                    most_ds = fmaxf(most_ds, fmaxf(fabsf(p[2 * j]), fabsf(p[2 * j + 1])));
                                    asm volatile("" : "+v"(p[2 * j]), "+v"(p[2 * j + 1]));
                                }
                                if constexpr (m == 1 && j < EARLY) dt.pair(j, p[2 * j], p[2 * j + 1]);
                                if constexpr (m == 2 && j < 4 && !HALVES) pt.pair(4 + j, p[8 + 2 * j], p[8 + 2 * j + 1]);
                            }
                        });
                        if constexpr (g == 3 * G - 1 && m == 2) {
                            if (__builtin_amdgcn_ballot_w64(most_ds > LARGEST)) {     // the same for its largest dS
                                most_ds = swap_halves_max(most_ds);
                                const int by = most_ds > LARGEST ? 127 + 11 - (int)(__float_as_uint(most_ds) >> 23) : 0;
                                fall -= by;
                                down = ldexpf(1.f, -fall);
#pragma unroll
                                for (int v = 0; v < 16; ++v) p[v] = ldexpf(p[v], by);
#pragma unroll
                                for (int j = 0; j < EARLY; ++j) dt.pair(j, p[2 * j], p[2 * j + 1]);
#pragma unroll
                                for (int d = 0; d < DT; ++d)
#pragma unroll
                                    for (int v = 0; v < 16; ++v) acc[1][d][v] = ldexpf(acc[1][d][v], by);
                            }
                        }
                    }
                    if constexpr (HALVES && g > 2 * G && g % 2 == 0 && m == 2) {      // the tile before is complete
                        constexpr int tile = (g - 2 * G) / 2 - 1;
                        acc[tile / DT][tile % DT] += part[tile % 2];
                    }
                });
            if constexpr (HALVES) acc[1][DT - 1] += part[(DT - 1) % 2];
            buf = next;
        }
        VMOBA_WAIT_VMCNT(0);
    }
    if constexpr (HALVES) {                                       // sums of wavefronts 2 and 3 to 0 and 1, at the lower of the two scales
        static_assert(2 * 2 * DT * 16 * 64 * 4 <= 4 * DkvSmem<D>::CHUNK, "they fit");
        __syncthreads();                                          // nothing is on its way to the LDS, nobody reads rows any more
        float* part = reinterpret_cast<float*>(sm.rows) + (wave & 1) * (2 * DT * 16 * 64) + lane;
        if (wave >= 2) {
            sm.ld[wave][lane] = __int_as_float(lift);
            sm.ld[wave - 2][lane] = __int_as_float(lift - fall);
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int d = 0; d < DT; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) part[((x * DT + d) * 16 + v) * 64] = acc[x][d][v];
        }
        __syncthreads();
        if (wave >= 2) return;
        const int mine[2] = {lift, lift - fall};
        int low[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int other = __float_as_int(sm.ld[wave + 2 - 2 * x][lane]);
            low[x] = min(mine[x], other);
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    acc[x][d][v] = ldexpf(acc[x][d][v], low[x] - mine[x]) + ldexpf(part[((x * DT + d) * 16 + v) * 64], low[x] - other);
        }
        lift = low[0];
        fall = low[0] - low[1];
    }
    if (kk < L) {
        const long long kout = rows ? rows[krow] : krow;
        float* pv = reinterpret_cast<float*>(dV.ptr + ((long long)run.b * dV.stride_b + kout * dV.stride_s + (long long)run.h * dV.stride_h) * 4);
        float* pk = reinterpret_cast<float*>(dK.ptr + ((long long)run.b * dK.stride_b + kout * dK.stride_s + (long long)run.h * dK.stride_h) * 4);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4_t ov, ok;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    ov[r] = ldexpf(acc[0][dt][4 * i + r], -(lift + pw.y));
                    ok[r] = ldexpf(acc[1][dt][4 * i + r] * scale, -(lift - fall + pw.y + pw.w + pw.x));
                }
                *reinterpret_cast<f32x4_t*>(pv + dt * 32 + i * 8 + hf * 4) = ov;
                *reinterpret_cast<f32x4_t*>(pk + dt * 32 + i * 8 + hf * 4) = ok;
            }
    }
}

template <int D>
__global__ __launch_bounds__(256, 1) void attn_bwd_dkv_split_kernel(
    const char* __restrict__ QD4, const char* __restrict__ KV4, const int4* __restrict__ power, const float* __restrict__ lse_delta, const int* __restrict__ blk_off,
    const int* __restrict__ blk_ptr, const int* __restrict__ q_idx, const int* __restrict__ kb_start, const int* __restrict__ kb_order,
    const int* __restrict__ out_of_range, TensorView dK, TensorView dV, const int* __restrict__ rows, int Hh, int S, int pitch, int nb, long long cap,
    float scale_log2, float scale, int BH, int slots, int group) {
    __shared__ DkvSmem<D> sm;
    if (*out_of_range) return;
    // groups of one block's runs to the XCDs in turn, heads inside a group number (see attn_bwd_dkv_kernel): 2.51 -> 2.22 ms
    const int n = (int)blockIdx.x >> 3, G = (n / group) * 8 + ((int)blockIdx.x & 7);
    if (G >= BH * (slots / group)) return;
    DkvRun run;
    run.bh = G % BH; run.b = run.bh / Hh; run.h = run.bh % Hh;
    const int run_id = (G / BH) * group + n % group;
    const int* ks = kb_start + (long long)run.bh * (nb + 1);
    int lo = 0, hi = nb;
    if (run_id >= ks[nb]) return;
    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (ks[mid] <= run_id) lo = mid; else hi = mid; }
    run.first = (run_id - ks[lo]) * 128;
    run.j = kb_order[(long long)run.bh * nb + lo];
    run.k0 = blk_off[run.j]; run.L = blk_off[run.j + 1] - run.k0;
    run.list0 = blk_ptr[(long long)run.bh * (nb + 1) + run.j];
    run.cnt = blk_ptr[(long long)run.bh * (nb + 1) + run.j + 1] - run.list0;
    const int* list = q_idx + (long long)run.bh * cap + run.list0;
    const int4 pw = power[run.bh];                                // of Q, dO, K, V
    if (run.L - run.first <= 64) dkv_run<D, true>(sm, run, QD4, KV4, pw, lse_delta, list, dK, dV, rows, S, pitch, scale_log2, scale);
    else dkv_run<D, false>(sm, run, QD4, KV4, pw, lse_delta, list, dK, dV, rows, S, pitch, scale_log2, scale);
}

}  // namespace

void launch_split_rows(int D, int BH, int Hh, int S, hipStream_t st, const SplitTensors& in, int n, void* scratch, int4** power, int* out_of_range) {
    const int chunks = split_scan_chunks(S);
    uint2* partial = (uint2*)((char*)scratch + (size_t)BH * 16);
    *power = (int4*)scratch;
    auto scan = D == 128 ? split_scan_kernel<128> : split_scan_kernel<64>;
    scan<<<dim3((unsigned)chunks, (unsigned)BH, (unsigned)n), dim3(256), 0, st>>>(in, partial, Hh, S);
    const dim3 grid((unsigned)ceil_div64(S, 4 * 256 / (D / 8)), (unsigned)BH, (unsigned)n);
    auto kfn = D == 128 ? split_rows_kernel<128> : split_rows_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(in, partial, chunks, (int*)*power, Hh, S, out_of_range);
}

void launch_fwd_tiles_split(int D, dim3 grid, hipStream_t st, const char* Q2, const char* KV4, const int4* power, const int* q_idx, const int4* flat_desc,
                            const int* n_tiles, const int* out_of_range, float* Opart, float* lse_part, int S, long long cap, float scale_log2) {
    auto kfn = D == 128 ? attn_fwd_tile_split_kernel<128> : attn_fwd_tile_split_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(Q2, KV4, power, q_idx, flat_desc, n_tiles, out_of_range, Opart, lse_part, S, cap, scale_log2);
}

void launch_dq_tiles_split(int D, dim3 grid, hipStream_t st, const char* QD4, const char* KV4, const int4* power, const float* lse_delta, const int* q_idx,
                           const int4* flat_desc, const int* n_tiles, const int* out_of_range, float* dQpart, int S, int pitch, long long cap,
                           float scale_log2) {
    auto kfn = D == 128 ? attn_bwd_dq_split_kernel<128> : attn_bwd_dq_split_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(QD4, KV4, power, lse_delta, q_idx, flat_desc, n_tiles, out_of_range, dQpart, S, pitch, cap, scale_log2);
}

void launch_dkv_split(int D, dim3 grid, hipStream_t st, const char* QD4, const char* KV4, const int4* power, const float* lse_delta, const int* blk_off,
                      const int* blk_ptr, const int* q_idx, const int* kb_start, const int* kb_order, const int* out_of_range, const TensorView& dK,
                      const TensorView& dV, const int* rows, int Hh, int S, int pitch, int nb, long long cap, float scale_log2, float scale, int BH, int slots,
                      int group) {
    auto kfn = D == 128 ? attn_bwd_dkv_split_kernel<128> : attn_bwd_dkv_split_kernel<64>;
    kfn<<<grid, dim3(256), 0, st>>>(QD4, KV4, power, lse_delta, blk_off, blk_ptr, q_idx, kb_start, kb_order, out_of_range, dK, dV, rows, Hh, S, pitch, nb,
                                    cap, scale_log2, scale, BH, slots, group);
}
