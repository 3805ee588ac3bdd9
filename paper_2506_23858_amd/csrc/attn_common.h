// Pieces shared by the forward and backward block-sparse attention kernels.
//
// Work decomposition (both directions).  The selection mask is kept block-major, the
// orientation M_i in (N_b, s) of Eq. 3: for key block j, q_idx[blk_ptr[j] .. blk_ptr[j+1]) lists
// the queries that keep it.  A "tile" is TM consecutive entries of one such list, i.e. TM gathered
// queries that all attend to the same key block.  The list of all heads' tiles is written on the
// device from blk_ptr, so the host never learns the data-dependent counts; the grid is sized from
// nnz_capacity and surplus workgroups leave at once.
//
// MFMA operand plumbing (v_mfma_f32_32x32x16_bf16; lane = 32*hf + l32):
//   A operand: lane holds row l32, 8 consecutive k at 8*hf;   B operand: column l32, same k.
//   C/D:       lane holds column l32, rows 8*i + 4*hf + r as value 4*i + r (i, r = 0..3).
// Row tiles in LDS are laid out as RowTile (below) says; the dK/dV kernel's body for short block tails pads its rows instead
// (row stride D + 8).
//   * An operand that contracts over the channels of a row is a 16-byte row read.
//   * An operand that contracts over the ROWS (the transposed tile) is two ds_read_b64_tr_b16:
//     in each group of 16 lanes, lane 4*e + a supplies the address of 4 consecutive channels of
//     one row and receives, for channel 4*a' + c of the group (lane = 4*a' + c), the values of
//     the 4 rows supplied by lanes a', a'+4, a'+8, a'+12.
//   * Rows are fed to the first MFMA through the bit permutation rho below.  With it the 8
//     accumulator values a lane holds per 16-row step belong to rows {16*s + 4*e + 2*t + hf},
//     e = 0..3, t = 0..1: they pack straight into the next MFMA's B operand (no shuffle), the
//     matching transposed A operand is exactly what the two transpose reads (t = 0, 1) deliver,
//     and both kinds of LDS access are bank-conflict free with either layout.
#pragma once
#include "common.h"

#include <type_traits>

// MFMA row m (0..31) of a 32-row group is fed tile row rho(m):
//   rho = 16*m[4] + 4*m[1:0] + 2*m[3] + m[2]
__device__ __forceinline__ int rho(int m) {
    return (m & 16) | ((m & 3) << 2) | ((m & 8) >> 2) | ((m & 4) >> 2);
}
// Tile row (0..31) that accumulator value v (0..15) of lane half hf belongs to.
__device__ __forceinline__ int acc_row(int v, int hf) {
    return ((v >> 3) << 4) | ((v & 3) << 2) | (((v >> 2) & 1) << 1) | hf;
}

typedef __bf16 __attribute__((address_space(3))) lds_bf16_t;
typedef bf16x4_t __attribute__((address_space(3))) lds_bf16x4_t;

// Per-lane element offset of the transposed-operand reads inside a tile of row stride STR:
// row 4*e + hf, channel 16*(g&1) + 4*a, with lane = 16*g + 4*e + a.
template <int STR>
__device__ __forceinline__ int tr_lane_offset(int lane) {
    const int g = lane >> 4, e = (lane >> 2) & 3, a = lane & 3, hf = lane >> 5;
    return (4 * e + hf) * STR + 16 * (g & 1) + 4 * a;
}

// Transposed A operand: m = channel col0 + l32, k-slots = rows {row0 + 16*s + 4*e + 2*t + hf}.
// `tile_lane` = tile base + tr_lane_offset (per lane); row0 = 32 * (row group), s = 16-row step.
template <int STR>
__device__ __forceinline__ bf16x8_t tr_operand(const __bf16* tile_lane, int row0, int s, int col0) {
    const __bf16* p = tile_lane + (row0 + 16 * s) * STR + col0;
    const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p));
    const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p + 2 * STR));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ bf16x8_t pack8(const float* p) {
    f32x4_t lo = {p[0], p[1], p[2], p[3]};
    f32x4_t hi = {p[4], p[5], p[6], p[7]};
    bf16x4_t blo = __builtin_convertvector(lo, bf16x4_t);
    bf16x4_t bhi = __builtin_convertvector(hi, bf16x4_t);
    return __builtin_shufflevector(blo, bhi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// f(0), f(1), ... f(N - 1) with the index as a compile-time constant.
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

struct Tile {
    int list0;    // first list entry of the tile, relative to the head's segment
    int count;    // valid entries in the tile (1..TM)
    int bh;       // batch element and head
    int k0, L;    // first key position and number of keys of the tile's key block
};
__device__ __forceinline__ Tile tile_of(const int4 d) { return {d.x, d.y & 1023, d.y >> 10, d.z, d.w}; }      // see write_tile_list
// The tile of a workgroup of a kernel with one workgroup per entry of the flat list (all heads); false: none.  Workgroup ids go round
// the 8 XCDs, so XCD x = id % 8 takes the x-th eighth of the list: a key block's tiles then share one L2 instead of eight
// (gridDim.x is a multiple of 8).
__device__ __forceinline__ bool take_tile(const int4* __restrict__ flat_desc, const int* __restrict__ n_tiles, Tile& t) {
    const int total = *n_tiles, per_xcd = (total + 7) >> 3, slot = (int)(blockIdx.x >> 3);
    const int f = (int)(blockIdx.x & 7) * per_xcd + slot;
    if (slot >= per_xcd || f >= total) return false;
    t = tile_of(flat_desc[f]);
    return true;
}

inline __device__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

// Sum over the workgroup's 256 threads of the values before this thread's (exclusive prefix sum); *total receives the sum
// of all.  sW: four words of LDS.  Contains two barriers.
__device__ __forceinline__ int block_exclusive_sum256(int v, int* sW, int* total) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    __syncthreads();
    if (lane == 63) sW[wv] = incl;
    __syncthreads();
    int base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wv) base += sW[w];
        sum += sW[w];
    }
    *total = sum;
    return base + incl - v;
}

// One workgroup's part of the flat tile list over all heads (heads in order, blocks in order): descriptors
// {first list entry, count | head << 10, first key, block length} of tiles tile0, tile0 + 1, ... tile0 + 255 of head bh, at
// flat_desc[tiles of the heads before + tile]; the last head's workgroups also write *n_tiles, the length of the list.
// Every workgroup counts the tiles of the heads before its own and scans its own head's blocks by itself -- at most some
// thousand cached loads -- so that the list takes one launch and no workgroup waits for another.  With so many heads that this
// would be the larger part (heads_counted_first), head_tiles holds every head's number of tiles, counted in a launch before.
struct TileListLds { int start[VMOBA_MAX_BLOCKS + 1]; int wave[4]; };
__device__ __forceinline__ void write_tile_list(TileListLds& lds, const int* __restrict__ blk_ptr, const int* __restrict__ blk_off,
                                                const int* __restrict__ head_tiles, int4* __restrict__ flat_desc, int* __restrict__ n_tiles, int bh, int BH,
                                                int nb, int TM, int tile0) {
    const int t = threadIdx.x;
    const int* bp = blk_ptr + (long long)bh * (nb + 1);
    int mine = 0;
    if (head_tiles) {
        for (int i = t; i < bh; i += 256) mine += head_tiles[i];
    } else {
        for (unsigned i = t; i < (unsigned)bh * nb; i += 256) {
            const unsigned hh = i / (unsigned)nb, j = i - hh * nb;
            const int* q = blk_ptr + (size_t)hh * (nb + 1) + j;
            mine += (q[1] - q[0] + TM - 1) / TM;
        }
    }
    int first;
    (void)block_exclusive_sum256(mine, lds.wave, &first);
    static_assert(VMOBA_MAX_BLOCKS <= 512, "two blocks per thread");
    int n0 = 0, n1 = 0, total;
    if (2 * t < nb) n0 = (bp[2 * t + 1] - bp[2 * t] + TM - 1) / TM;
    if (2 * t + 1 < nb) n1 = (bp[2 * t + 2] - bp[2 * t + 1] + TM - 1) / TM;
    const int excl = block_exclusive_sum256(n0 + n1, lds.wave, &total);
    if (2 * t < nb) lds.start[2 * t] = excl;
    if (2 * t + 1 < nb) lds.start[2 * t + 1] = excl + n0;
    if (t == 0) {
        lds.start[nb] = total;
        if (bh == BH - 1 && tile0 == 0) *n_tiles = first + total;
    }
    __syncthreads();
    const int tile = tile0 + t;
    if (tile >= total) return;
    int lo = 0, hi = nb;           // largest j with start[j] <= tile
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (lds.start[mid] <= tile) lo = mid; else hi = mid;
    }
    const int t0 = (tile - lds.start[lo]) * TM;
    const int e0 = bp[lo] + t0, k0 = blk_off[lo];
    flat_desc[first + tile] = make_int4(e0, min(TM, bp[lo + 1] - e0) | (bh << 10), k0, blk_off[lo + 1] - k0);
}
// Blocks of all heads from which on they are counted first.  Forward + backward calls without / with the launch, us: 2000 blocks 141 / 141,
// 10 240 (640 heads x 16) 434 / 414, (80 x 128) 591 / 575, 20 480 (1280 x 16) 883 / 827, 163 840 (10 240 x 16) 9466 / 7095.
static inline bool heads_counted_first(int BH, int nb) { return (int64_t)BH * nb > 8192; }
void launch_head_tiles(hipStream_t st, const int* blk_ptr, int* head_tiles, int BH, int nb, int TM);
// Grid of a kernel with one workgroup per entry of the flat list: a bound on its length, a multiple of 8.
static inline dim3 flat_tile_grid(int BH, int64_t max_tiles, int64_t cap, int TM, int nb) {
    const int64_t a = (int64_t)BH * max_tiles, b = ((cap / TM + nb) * (int64_t)BH + 15) / 8 * 8;
    return dim3((unsigned)(a < b ? a : b));
}
// Pitch of the LSE * log2(e) and -delta arrays the backward kernels read, [head][2][pitch]: element S of either is what a row past
// the end of a query list reads (LSE +inf, i.e. weight 0, and delta 0).
__host__ __device__ constexpr int lse_delta_pitch(int S) { return (S + 64) / 64 * 64; }

// float32 tile kernels (attn_f32.hip).  run_if: null, or a flag on the device without which they leave at once.
void launch_fwd_tiles_f32(int D, dim3 grid, hipStream_t st, const int* run_if, const TensorView& Q, const TensorView& K, const TensorView& V, const int* q_idx,
                          const int4* flat_desc, const int* n_tiles, float* Opart, float* lse_part, int Hh, long long cap,
                          float scale_log2, const int* kv_rows);
void launch_dq_tiles_f32(int D, dim3 grid, hipStream_t st, const int* run_if, const TensorView& Q, const TensorView& K, const TensorView& V, const TensorView& dO,
                         const float* lse_delta, const int* q_idx, const int4* flat_desc, const int* n_tiles,
                         float* dQpart, int Hh, int S, long long cap, float scale_log2, const int* kv_rows);
// parts: 64-key parts per entry of the run table (1, or 2 where the table counts runs of 128 keys)
void launch_dkv_f32(int D, dim3 grid, hipStream_t st, const int* run_if, int parts, const TensorView& Q, const TensorView& K, const TensorView& V, const TensorView& dO,
                    const float* lse_delta, const int* blk_off, const int* blk_ptr, const int* q_idx, const int* kb_start,
                    const int* kb_order, const TensorView& dK, const TensorView& dV, const int* rows, int Hh, int S, int nb, long long cap,
                    float scale_log2, float scale, const int* kv_rows);
// The same on the bfloat16 matrix instruction, from rows split into three terms each (attn_split.hip).
void launch_split_rows(int D, int BH, int Hh, int S, hipStream_t st, const TensorView& X, const int* map, char* dst, int planes, int plane0, int* out_of_range);
void launch_fwd_tiles_split(int D, dim3 grid, hipStream_t st, const char* Q3, const char* KV6, const int* q_idx, const int4* flat_desc,
                            const int* n_tiles, const int* out_of_range, float* Opart, float* lse_part, int S, long long cap, float scale_log2);
void launch_dq_tiles_split(int D, dim3 grid, hipStream_t st, const char* QD6, const char* KV6, const float* lse_delta, const int* q_idx,
                           const int4* flat_desc, const int* n_tiles, const int* out_of_range, float* dQpart, int S, int pitch, long long cap,
                           float scale_log2);
void launch_dkv_split(int D, dim3 grid, hipStream_t st, const char* QD6, const char* KV6, const float* lse_delta, const int* blk_off, const int* blk_ptr,
                      const int* q_idx, const int* kb_start, const int* kb_order, const int* out_of_range, const TensorView& dK, const TensorView& dV,
                      const int* rows, int Hh, int S, int pitch, int nb, long long cap, float scale_log2, float scale, int BH, int slots, int group);
// float32 calls with enough work -- multiply-adds of one product over all pairs the lists can hold -- take the split kernels, if
// 32-bit offsets reach every split row of a head.  What they cost beside their products is seven passes over the inputs
// and ten launches in a training step; what they save grows with the pairs and with the length of the blocks (below some 64 keys
// the partial rows set the time).  Training step (forward) with / without them, us: blocks of 300 keys, work 6.7e7:
// 207 / 251 (95 / 107), 2.4e9: 421 / 613 (153 / 176); 128 keys, 3.0e8: 210 / 212; 64 keys, 3.0e8: 225 / 228 (98 / 97), 2.4e9: 538 / 570
// (205 / 217); 32 keys, 3.0e8: 263 / 255, 2.4e9: 880 / 936 (298 / 287).
static inline bool use_split(int BH, int64_t S, int D, int n_blocks, int64_t cap) {
    const double len = (double)S / n_blocks, work = (double)BH * (double)cap * (double)D * len;
    return work * (len / 128) * (len / 128) >= 2e8 && S < (1 << 24) && (uint64_t)S * 12 * (uint64_t)D < ((uint64_t)1 << 32);
}
// Compute units of the current device (queried once).
int vmoba_num_cus();

// Exchange between the two halves of a wavefront (lane i <-> lane i ^ 32), reduced with max / sum.
__device__ __forceinline__ float swap_halves_max(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ float swap_halves_sum(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}
// 64 lanes x 16 bytes from base + byte_off (per lane) to LDS: lane i writes lds_addr + 16 * i (lds_addr is
// wave-uniform).  Counts in vmcnt like any vector load; the compiler does not know about it.
__device__ __forceinline__ void dma16(const char* base, uint32_t byte_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr)
                 : "memory", "m0");
}
// The same to lds_addr + lds_off, and next += advance: m0 may not be read right after it was written, so the addition stands between, and
// byte_off, read behind it, may not share next's register (&).
__device__ __forceinline__ void dma16_advance(const char* base, uint32_t byte_off, uint32_t& next, uint32_t advance, uint32_t lds_addr, uint32_t lds_off) {
    asm volatile("s_add_u32 m0, %3, %4\n\tv_add_u32 %0, %5, %0\n\tglobal_load_lds_dwordx4 %1, %2"
                 : "+&v"(next) : "v"(byte_off), "s"(base), "s"(lds_addr), "s"(lds_off), "s"(advance) : "memory", "m0", "scc");
}
// The same from any address per lane.
__device__ __forceinline__ void dma16_at(const char* src, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}
// The same with 4 bytes per lane: lane i writes lds_addr + 4 * i.
__device__ __forceinline__ void dma4(const char* base, uint32_t byte_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(byte_off), "s"(base), "s"(lds_addr)
                 : "memory", "m0");
}
#define VMOBA_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// ---------------------------------------------------------------------------------------------
// Rows of Q, K, V and dO go from global memory to LDS without passing through registers (global_load_lds, inline assembly, waits
// written by hand): the 64 lanes of one request write 1024 consecutive bytes, i.e. RPI = 4 (8) rows of D = 128 (64) channels.
// Such groups of rows lie GP bytes apart, and 16-byte piece p of a group's row i sits at piece position p ^ fsw(i).  Row and
// transposed reads are then free of bank conflicts, and for D = 128 only the two low bits of a piece position depend on the
// row, so that two per-lane addresses and immediate offsets reach every operand of a tile.
template <int D>
struct RowTile {
    static constexpr int RB = 2 * D, PPR = D / 8, RPI = 64 / PPR;
    static constexpr int GP = D == 128 ? 1024 + 64 : 1024 + 144;       // bytes between groups of RPI rows
    static constexpr int HB = 32 / RPI * GP;                           // bytes of 32 rows
    static constexpr int DT = D / 32;
    static constexpr int NRB = D == 128 ? 2 : 4;                       // distinct per-lane addresses of the row reads
    static constexpr int NTB = D == 128 ? 1 : DT;                      // and, for each half, of the transposed reads
    __device__ static __forceinline__ int fsw(int i) { return D == 128 ? i : 2 * ((i >> 1) & 1) + 4 * (i >> 2); }
    // byte offset inside a row that lane `lane` of a request fetches
    __device__ static __forceinline__ uint32_t request_piece(int lane) { return (uint32_t)((lane % PPR) ^ fsw(lane / PPR)) * 16; }
    // Per-lane addresses of the operands of a 32-row tile: contraction over the channels (row rho(l32), k-step ks) ...
    __device__ static __forceinline__ uint32_t row_lane(int lane, int ks) {
        const int r = rho(lane & 31), hf = lane >> 5;
        return (uint32_t)(r / RPI * GP + r % RPI * RB + ((2 * ks + hf) ^ fsw(r % RPI)) * 16);
    }
    // ... and over the rows (see tr_lane_offset; half t of the operand, channel tile dt)
    __device__ static __forceinline__ uint32_t tr_lane(int lane, int t, int dt) {
        const int g4 = lane >> 4, e = (lane >> 2) & 3, a = lane & 3, hf = lane >> 5;
        const int r = 4 * e + hf + 2 * t;
        return (uint32_t)(r / RPI * GP + r % RPI * RB + ((4 * dt + 2 * (g4 & 1) + (a >> 1)) ^ fsw(r % RPI)) * 16 + (a & 1) * 8);
    }
    // Operands at byte offset `tile` of `base`; rl = row_lane(., 0 .. NRB - 1), tl = tr_lane(., 0 .. 1, 0 .. NTB - 1)
    __device__ static __forceinline__ bf16x8_t rows(const char* base, const uint32_t* rl, uint32_t tile, int ks) {
        return *reinterpret_cast<const bf16x8_t*>(base + (rl[ks % NRB] + tile) + (ks / NRB) * 64);
    }
    __device__ static __forceinline__ bf16x8_t transposed(const char* base, const uint32_t (*tl)[NTB], uint32_t tile, int s, int dt) {
        bf16x4_t h[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
            h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                (lds_bf16x4_t*)(base + (tl[t][NTB == 1 ? 0 : dt] + tile) + s * (16 / RPI) * GP + (NTB == 1 ? dt * 64 : 0)));
        return __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    }
};

// The same for v_mfma_f32_16x16x32_bf16 (lane = 16 * g + l16): A operand: lane holds row l16, 8 consecutive k at 8 * g; B operand: column
// l16, same k; C/D: lane holds column l16, rows 4 * g + i as value i.  Rows are fed in their order: the accumulators of two 16-row
// tiles, rows 4 * g + i and 16 + 4 * g + i, pack straight into the next product's B operand of 32 rows, and two transpose reads deliver
// the A operand that goes with it.  (The 16-row instruction does the same work in the same cycles with half the traffic of sums: under the
// card's power limit a loop of nothing else runs at 2.05 PFLOP/s, 2.0 GHz, against 1.79, 1.75 GHz, of the 32-row one.)
// Rows lie one after the other, row r's 16-byte piece p at piece position p ^ swz(r).  The LDS serves 256 bytes per cycle: 16 lanes of a
// row read (eight rows of one piece, the other eight of the next: lanes 0-3, 12-15, 20-23 and 24-27, and so on) have to hit 16 different
// pieces of 256 bytes, and the 32 lanes of a transposed read (8 rows of two pieces) as well.  So swz leaves the lowest bit alone and is one-to-one
// in the others over 8 rows (D = 64: over the 4 of either parity, which share no piece positions).
template <int D>
struct RowTile16 {
    static constexpr int RB = 2 * D, PPR = D / 8, RPI = 64 / PPR;
    static constexpr int HB = 32 * RB;                                 // bytes of 32 rows
    static constexpr int NPC = 8 / RPI;                                // different requests, see request_piece
    static constexpr int NRB = D / 32, NTB = D / 16;                   // per-lane addresses of the row and of the transposed reads
    __device__ static __forceinline__ int swz(int r) { return D == 128 ? (r & 7) << 1 : (r & 6); }
    // byte offset inside a row that lane `lane` of the request for rows RPI * j ... fetches (j modulo NPC)
    __device__ static __forceinline__ uint32_t request_piece(int lane, int j) { return (uint32_t)((lane % PPR) ^ swz(RPI * j + lane / PPR)) * 16; }
    // contraction over the channels: row l16, k-step ks of 32 channels ...
    __device__ static __forceinline__ uint32_t row_lane(int lane, int ks) {
        return (uint32_t)((lane & 15) * RB + ((4 * ks + (lane >> 4)) ^ swz(lane & 15)) * 16);
    }
    // ... and over the rows: channel tile ct of 16; lane = 16 * g + 4 * e + a asks for four channels of row 4 * g + e
    __device__ static __forceinline__ uint32_t tr_lane(int lane, int ct) {
        const int r = lane >> 2, a = lane & 3;
        return (uint32_t)(r * RB + ((2 * ct + (a >> 1)) ^ swz(r)) * 16 + (a & 1) * 8);
    }
    // Operands at byte offset `tile` of `base`; rl = row_lane(., 0 .. NRB - 1), tl = tr_lane(., 0 .. NTB - 1); kt: 16-row half of the 32 rows
    __device__ static __forceinline__ bf16x8_t rows(const char* base, const uint32_t* rl, uint32_t tile, int kt, int ks) {
        return *reinterpret_cast<const bf16x8_t*>(base + (rl[ks] + tile) + kt * 16 * RB);
    }
    __device__ static __forceinline__ bf16x8_t transposed(const char* base, const uint32_t* tl, uint32_t tile, int ct) {
        bf16x4_t h[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(base + (tl[ct] + tile) + t * 16 * RB));
        return __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
    }
};

// 64 lanes x 16 bytes, row `row` of a matrix of `stride` bytes per row (both below 2^24), byte `piece` of it, to LDS lds + IMM.
template <int IMM>
__device__ __forceinline__ void dma_row16(const char* base, uint32_t row, uint32_t stride, uint32_t piece, uint32_t lds) {
    uint32_t off;
    asm volatile("s_add_u32 m0, %5, %6\n\tv_mad_u32_u24 %0, %1, %2, %3\n\tglobal_load_lds_dwordx4 %0, %4"
                 : "=&v"(off) : "v"(row), "s"(stride), "v"(piece), "s"(base), "s"(lds), "i"(IMM) : "memory", "m0", "scc");
}
