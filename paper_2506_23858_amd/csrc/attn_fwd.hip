// vmoba_attn_fwd: Step 3 of Sec. 3.1 -- every query attends to the keys/values of its selected
// blocks only.
//
// Two phases.  (1) Tile kernel, block-major: a workgroup takes TM gathered queries of one key
// block j and runs flash-attention (online soft-max) over the L_j keys of that block alone,
// writing a normalised partial output and its log-sum-exp per (query, block) pair.  (2) Merge
// kernel, query-major: the partials of a query's selected blocks are combined with weights
// exp(lse_pair - LSE).  bfloat16 inputs use the 32x32x16 bf16 MFMA; the tile kernel for float32
// inputs is in attn_f32.hip.
#include "attn_common.h"

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// The flat tile list of a forward call (see write_tile_list); grid: 256 tile ids x head.
__global__ __launch_bounds__(256) void tile_list_kernel(const int* __restrict__ blk_ptr, const int* __restrict__ blk_off,
                                                        const int* __restrict__ head_tiles, int4* __restrict__ flat_desc, int* __restrict__ n_tiles, int* __restrict__ clear,
                                                        int BH, int nb, int TM) {
    __shared__ TileListLds lds;
    if (clear && (blockIdx.x | blockIdx.y | threadIdx.x) == 0) *clear = 0;
    write_tile_list(lds, blk_ptr, blk_off, head_tiles, flat_desc, n_tiles, blockIdx.y, BH, nb, TM, blockIdx.x * 256);
}

// head_tiles[h] = number of tiles of head h; one wavefront per head.
__global__ __launch_bounds__(256) void head_tiles_kernel(const int* __restrict__ blk_ptr, int* __restrict__ head_tiles, int BH, int nb, int TM) {
    const int h = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (h >= BH) return;
    const int* bp = blk_ptr + (long long)h * (nb + 1);
    int n = 0;
    for (int j = lane; j < nb; j += 64) n += (bp[j + 1] - bp[j] + TM - 1) / TM;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off, 64);
    if (lane == 0) head_tiles[h] = n;
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA tile kernel.  NW wavefronts; wavefront w owns 32 gathered queries (a tile is 32 * NW list
// entries of one key block) and the block's keys are walked in groups of 32.
//
// Operand orientation.  All products are computed transposed so that the query index is the MFMA
// column (= lane % 32):
//   S^T[key, q] = K[key, :] . Q[q, :]          A = K rows from LDS, B = Q^T held in registers
//   O^T[d, q]  += V^T[d, key] . P^T[key, q]    A = V^T by transpose reads, B = P^T packed from S^T
// With the query on the lane, the row maximum and row sum of the online soft-max are reductions
// over a lane's own registers plus one exchange between the lane halves (v_permlane32_swap).
//
// One stream of key groups.  A workgroup is persistent: it strides through its XCD's share of the flat tile list (all heads,
// see write_tile_list), and the key groups of its tiles form one sequence that is worked on without a break.  Step n of a wavefront,
// a three-stage software pipeline, issues
//     S^T(n+1) = K(n+1) . Q^T               (matrix)
//     P(n)     = soft-max piece of S^T(n)   (vector)
//     O^T     += V(n-1)^T . P(n-1)^T        (matrix)
// unit by unit (unit u = k-step u of the first product and (s, dt) = (u / DT, u % DT) of the second), with the LDS operands
// of unit u + 2 fetched during unit u, so neither LDS latency nor the soft-max sits between dependent matrix instructions.
// S^T and P live in two register sets that swap roles every step.  A tile's last step computes S^T of the next tile's first group, and the
// next tile's first step ends the tile's second product: no steps with half of the work missing at a tile's ends.  A tile
// counts as at least four groups (surplus ones are masked like the keys past a block's end), which is what the look-ahead of the
// row requests needs.  The value rows of a group without a key are zeros: repeating the block's last row would turn an infinity in it into weight 0
// times infinity, which is no number.
//
// What bounds it: two wavefronts of a SIMD together issue one instruction, scalar ones and waits included, every 4.5 cycles or so, and the clock
// falls as the rate rises (1.8 GHz here, 2.4 without load).  A step is 150 instructions for 16 matrix instructions (165 before): row
// offsets advance in the request itself, ring slots change names, and everything that only happens at a tile's ends stays out of the
// steps between.  With the steps at a tile's ends gone as well, the kernel takes, before -> after, at 480p, 12 heads, 1D / 2D / 3D with keys
// in place (and tau = 0.5): 1.34 / 1.42 / 2.65 -> 1.26 / 1.26 / 2.49 ms; at 720p, 10 of 40 blocks per query, 8.5 -> 8.0 ms.  Timing variants:
// no LDS operand reads -12 %, no exponentials -15 %, no row requests -10 %, the barrier in every second step only -3 %.
//
// Rows.  K and V groups are loaded straight from global memory into rings of four LDS slots each
// (global_load_lds_dwordx4: 64 lanes x 16 bytes land in 1024 consecutive LDS bytes), so no
// registers hold rows in flight.  A slot is a 32-row RowTile: two per-lane addresses and immediate offsets reach every operand.
// Rows past the end of the block repeat its last key; the surplus keys of the last group are masked to -inf in the soft-max.
// The next tile's query rows go the same way, into the place of the partial rows, from where the Q^T registers are filled in the
// last step but one; their list entries, one tile earlier, into a small ring, and the descriptor another tile earlier.
//
// Soft-max.  The running maximum is only raised when a group exceeds it by more than 2^8 (the probabilities then
// stay below 2^8, well inside float32 / bf16 range), so that a step only compares its largest score with a limit and the rescaling is
// rare; the final division by the row sum makes the result independent of which maximum was used.  The row sum is
// kept per lane half and the halves are added once at the end (they always agree on the maximum).
//
// Ordering.  The loads are issued by inline assembly, so their waits are written by hand: a step starts with a wait for what this
// wavefront requested up to two steps before -- loads and stores count down in order, and all wavefronts issue the same
// sequence of them -- followed by the workgroup barrier, which makes everybody's rows visible.  Step n requests K(n+4) into the
// slot of K(n) (last read in step n-1) and V(n+2) into the slot of V(n-2) (last read in step n-1); K(n+2) and V(n) are first
// read at the end of step n.  The barrier is the bare instruction: operands on their way from LDS across it lie in slots that
// are not requested again before the step after, which cannot begin before they have been used.
//
// Output.  In the step after a tile's last a wavefront writes its 32 partial rows to LDS as the accumulators hold them (8 bytes
// per lane and channel group) and reads them back as whole rows: the tile's partials are
// consecutive rows of Opart, so each store request is a 1 KB run instead of 16-byte pieces of 32
// rows (the address unit needs about as long for one such request as for eight full-row ones).  Surplus rows of a tile repeat its
// last entry bit for bit and are stored to its place, so that every wavefront issues the same number of stores.
//
// Keys in place (KVR).  K and V may stay where the caller has them: key position p of the block order is then row
// kv_rows[p] of both.  The row numbers come by way of LDS, too (global_load_lds_dword): those of group g + 8 are requested
// in step g by every wavefront, those of a tile's first groups two tiles ahead, two groups by a wavefront, and a row request takes its row
// number from there one step before it is issued.  A tile's last steps still request the numbers of groups past its end, into its own
// ring, and those of the very last step may be on their way while the next tile's first step is worked on.  So that step fills a ring of which
// no tile in sight nor the tile just ended has a share: four rings, tile t in ring t % 4.  (tests/test_forward_schedule.py plays
// requests, waits and barriers and finds two requests for the same words that nothing orders, with three rings, and none with four.)
//
// NEG: the scores of -Q, for a negative scale (the scale given is its magnitude).
//
// SHORT: the products and the soft-max of groups without a key are left out, by tests in every unit of a tile's first two and last two
// steps.  For calls whose usual block has at most 64 keys (SHORT_BLOCK), so that two of four groups and more have none: without it such calls are
// bound by steps that do nothing.  (With a negative scale they stay so.)  Forward calls of 12 heads x 128 channels with blocks of 8 / 32 / 64 / 128 keys (480, 480, 256, 128 of them, tau = 0.25):
// 585 / 2708 / 1670 / 895 us without it, 560 / 2547 / 1596 / 920 with it; 16 heads x 64: 487 / 2200 / 1332 / 697 and 448 / 2025 / 1259 / 721.  In between, with
// 78 and 96 keys, large calls gain 1 to 2 % and small ones lose 2 %: 1560 tokens in blocks of 78, 41.2 and 42.1 us.
constexpr int SHORT_BLOCK = 64;
__device__ const u32x4_t zero_row[16] = {};        // one row of 128 channels
struct FwdArgs {
    TensorView Q, K, V;
    const int* q_idx;
    const int4* flat_desc;
    const int* n_tiles;
    float *Opart, *lse_part;
    long long cap;
    const int* kv_rows;
    int Hh;
    float scale_log2;
    int q_offsets_32;      // a row of Q is reached from its head by a 32-bit offset, a product of two numbers below 2^24
};
template <int D, int NW, bool KVR, bool NEG, bool SHORT>
__global__ __launch_bounds__(64 * NW, 8 / NW) void attn_fwd_tile_mfma_kernel(FwdArgs by_value) {
    // What is only needed at a tile's ends is read from the arguments again each time: there are not enough scalar registers to keep it.
    auto args = [&]() {
        auto p = (const __attribute__((address_space(4))) FwdArgs*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return p;
    };
    const int* const n_tiles = by_value.n_tiles;
    const float scale_log2 = by_value.scale_log2;
    const int* const kv_rows = by_value.kv_rows;
    constexpr int G = 32;                   // keys per group
    using TL = RowTile<D>;
    constexpr int PPR = TL::PPR;            // 16-byte pieces per row
    constexpr int SLOT = TL::HB;            // bytes per ring slot
    constexpr int NR = 4;                   // ring slots per tensor
    constexpr int KSTEPS = D / 16, DT = D / 32, UNITS = KSTEPS;
    constexpr int RPI = TL::RPI;            // rows per load instruction
    static_assert(G == RPI * NW, "one load instruction per wavefront, tensor and group");
    static_assert(UNITS % 4 == 0 && UNITS == 2 * DT && (D == 64 || D == 128), "unit bookkeeping");
    constexpr int MIN_GROUPS = 4;           // groups a tile counts as, at least
    const float lazy = 8.f / scale_log2;    // a row's maximum is raised by more than 2^8 only
    // the partial rows of a wavefront: 32 rows, written 8 bytes per lane and channel group, read back as whole rows
    constexpr int OPITCH = D * 2 + 16;
    constexpr int V0 = NR * SLOT, OUT0 = 2 * NR * SLOT, OUTW = 32 * OPITCH, IDX0 = OUT0 + NW * OUTW, DESC0 = IDX0 + 2 * NW * 64 * 4,
                  TOK0 = DESC0 + NW * 64 * 4;
    // KVR: row numbers of the key groups of the tile before, of this one and of the next two, rings of 16 groups (a request fills two)
    constexpr int ROW_RINGS = 4, TOKS = 17 * G;
    __shared__ __align__(1024) char smem[TOK0 + (KVR ? ROW_RINGS * TOKS * 4 : 0)];
    // requests and stores of a wavefront, always in this order: every step the rows of K and V (KVR: and row numbers); then, in a tile's
    // first step, (KVR: row numbers,) the partial rows and LSE of the tile before, a descriptor, list entries, query rows
    constexpr int N_STEP = KVR ? 3 : 2, N_FIRST = (KVR ? 1 : 0) + D * 2 * 32 / 1024 + 1 + 2 + 32 / RPI;
    static_assert(N_STEP + N_FIRST < 64, "what the wait counter holds");

    // Workgroup ids go round the 8 XCDs (each with its own L2), so XCD x = id % 8 takes the x-th eighth of the tile
    // list and its workgroups stride through it: a key block's tiles then share one L2 instead of eight.
    const int total = *n_tiles;
    const bool by_xcd = (gridDim.x & 7) == 0;
    const int xcd = by_xcd ? (int)(blockIdx.x & 7) : 0;
    const int f_step = by_xcd ? (int)(gridDim.x >> 3) : (int)gridDim.x;
    const int per_xcd = by_xcd ? (total + 7) >> 3 : total;
    const int f_end = min(total, (xcd + 1) * per_xcd);
    const int f0 = xcd * per_xcd + (by_xcd ? (int)(blockIdx.x >> 3) : (int)blockIdx.x);
    if (f0 >= f_end) return;
    int tiles_left = (f_end - f0 + f_step - 1) / f_step;             // tiles whose partial rows are still to be written
    const int f_last = f0 + (tiles_left - 1) * f_step;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hf = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const uint32_t lds_rows = lds0 + (uint32_t)wave * TL::GP;         // this wavefront's share of ring slot 0 of K
    char* const mine = smem + OUT0 + wave * OUTW;                     // this wavefront's partial rows, or next query rows
    const uint32_t lds_mine = lds0 + OUT0 + (uint32_t)wave * OUTW;

    struct FwdTile {
        int L, count, k0, bh;
        long long pair;                    // its first list entry, which is the first row of its partials, too
        const char *q, *k, *v;             // the head's rows
    };
    auto make_tile = [&](int4 d, const FwdTile& before) {            // (consecutive tiles mostly are the same head's)
        const Tile c = tile_of(d);
        FwdTile t = before;
        t.L = c.L;
        t.count = c.count;
        t.k0 = c.k0;
        t.bh = c.bh;
        const auto a = args();
        t.pair = (long long)c.bh * a->cap + c.list0;
        if (__builtin_expect(c.bh != before.bh, 0)) {
            const int b = c.bh / a->Hh, h = c.bh - b * a->Hh;
            t.q = a->Q.ptr + (b * a->Q.stride_b + h * a->Q.stride_h) * 2;
            t.k = a->K.ptr + (b * a->K.stride_b + h * a->K.stride_h) * 2;
            t.v = a->V.ptr + (b * a->V.stride_b + h * a->V.stride_h) * 2;
        }
        return t;
    };
    auto tile_at = [&](int f, const FwdTile& before) {
        const u32x4_t d = ((const __attribute__((address_space(4))) u32x4_t*)(uintptr_t)args()->flat_desc)[f];
        return make_tile(make_int4((int)d.x, (int)d.y, (int)d.z, (int)d.w), before);
    };
    auto groups_of = [&](const FwdTile& t) { return max((t.L + G - 1) / G, MIN_GROUPS); };
    // past the end of the workgroup's tiles: the last one again (its loads only)
    auto request_descriptor = [&](int f) {
        dma4(reinterpret_cast<const char*>(args()->flat_desc + min(f, f_last)), (uint32_t)min(lane, 3) * 4, lds0 + DESC0 + (uint32_t)wave * 256);
    };

    // list entries of the wavefront's queries (surplus rows repeat the tile's last query): tile's ring half `par`
    auto request_entries = [&](const FwdTile& t, int par) {
        dma4(reinterpret_cast<const char*>(args()->q_idx + t.pair), (uint32_t)min(wave * 32 + l32, t.count - 1) * 4, lds0 + IDX0 + (uint32_t)(par * NW + wave) * 256);
    };
    // The wavefront's 32 query rows, whole rows; piece p of row r sits at slot p ^ (r % pieces), which keeps the fragment reads free of
    // bank conflicts.  A wavefront reads back only what it requested: no barrier.
    auto request_queries = [&](const FwdTile& t, int par) {
        const auto a = args();
        const int* e = reinterpret_cast<const int*>(smem + IDX0) + (par * NW + wave) * 64 + lane / PPR;
        auto piece = [&](int k) { return (uint32_t)(((lane % PPR) ^ ((k * RPI + lane / PPR) & (PPR - 1))) * 16); };
        if (__builtin_expect(a->q_offsets_32, 1)) {
            static_for<32 / RPI>([&](auto k) {
                constexpr int k_ = decltype(k)::value;
                dma_row16<k_ * 1024>(t.q, (uint32_t)e[k_ * RPI], (uint32_t)(a->Q.stride_s * 2), piece(k_), lds_mine);
            });
        } else {
#pragma unroll
            for (int k = 0; k < 32 / RPI; ++k) dma16_at(t.q + e[k * RPI] * (a->Q.stride_s * 2) + piece(k), (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_mine + k * 1024));
        }
    };
    bf16x8_t qf[KSTEPS];
    auto read_query = [&](int ks) {
        u32x4_t x = *reinterpret_cast<const u32x4_t*>(mine + l32 * TL::RB + ((2 * ks + hf) ^ (l32 & (PPR - 1))) * 16);
        if constexpr (NEG) x ^= 0x80008000u;
        qf[ks] = __builtin_bit_cast(bf16x8_t, x);
    };

    // Row requests: row `dr` of a group is this lane's.  Byte offsets from the head's base are 32-bit (checked on the host); an offset past
    // the block's last row is clamped to it.
    const uint32_t pc16 = TL::request_piece(lane);
    const int dr = wave * RPI + lane / PPR;
    const uint32_t kss = (uint32_t)(by_value.K.stride_s * 2), vss = (uint32_t)(by_value.V.stride_s * 2);
    const uint32_t k_adv = G * kss, v_adv = G * vss;
    uint32_t krow = 0, vrow = 0;           // KVR: rows of the next request of K and of V, read from the ring a step before
    const char *k_base, *v_base;
    uint32_t k_off = 0, v_off = 0, k_last = 0, v_last = 0;
    auto begin_k = [&](const FwdTile& t) {
        k_base = t.k;
        k_off = (uint32_t)(t.k0 + dr) * kss + pc16;
        k_last = (uint32_t)(t.k0 + t.L - 1) * kss + pc16;
    };
    auto begin_v = [&](const FwdTile& t) {
        v_base = t.v;
        v_off = (uint32_t)(t.k0 + dr) * vss + pc16;
        v_last = (uint32_t)(t.k0 + t.L - 1) * vss + pc16;
    };
    // the next value rows requested, for a group without a key, are zeros (until begin_v)
    auto zero_v = [&]() {
        v_base = reinterpret_cast<const char*>(zero_row);
        v_off = v_last = pc16;
        vrow = 0;
    };
    // KVR: row numbers of groups x and x + 1 of tile t into ring `tb` (keys past the block's end repeat its last one)
    auto request_row_numbers = [&](const FwdTile& t, int x, int tb) {
        dma4(reinterpret_cast<const char*>(kv_rows), (uint32_t)(t.k0 + min(x * G + lane, t.L - 1)) << 2,
             lds0 + TOK0 + (uint32_t)(tb * TOKS + (x & 15) * G) * 4);
    };
    // groups 0..7, two per wavefront (with eight wavefronts, by two each: all issue the same number of requests)
    auto request_first_row_numbers = [&](const FwdTile& t, int tb) { request_row_numbers(t, 2 * (wave & 3), tb); };
    // KVR: row of K and V that this lane requests of group x of the tile of ring `tb`
    auto row_number = [&](int x, int tb) { return (uint32_t) reinterpret_cast<const int*>(smem + TOK0)[tb * TOKS + (x & 15) * G + dr]; };
    uint32_t rlane[TL::NRB], tlane[2][TL::NTB];
#pragma unroll
    for (int k = 0; k < TL::NRB; ++k) rlane[k] = TL::row_lane(lane, k);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int dt = 0; dt < TL::NTB; ++dt) tlane[t][dt] = V0 + TL::tr_lane(lane, t, dt);
    // Ring offsets of the slots n, n + 1, n + 2, n + 3 of the step n to come: they change places every step.
    uint32_t r0 = 0, r1 = SLOT, r2 = 2 * SLOT, r3 = 3 * SLOT;
    auto readK = [&](uint32_t off, int ks) { return TL::rows(smem, rlane, off, ks); };
    // transposed operand: channel tile dt = u % DT, 16-row step s = u / DT
    auto readV = [&](uint32_t off, int u) { return TL::transposed(smem, tlane, off, u / DT, u % DT); };
    const f32x16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    // ---- the first tile's rows: nothing to overlap them with
    int f_next = f0 + 3 * f_step;
    FwdTile none{};
    none.bh = -1;
    FwdTile cur = tile_at(f0, none), nxt = tile_at(min(f0 + f_step, f_last), cur), nn = tile_at(min(f0 + 2 * f_step, f_last), nxt);
    long long out_pair = 0;                // first pair and last entry of the tile before `cur`
    int out_last = -1;                     // -1: there is none
    int par = 0, tp = 0;                   // list-entry ring half and row-number ring of `cur`
    auto ring_ahead = [&](int tiles) { return (tp + tiles) & (ROW_RINGS - 1); };
    request_entries(cur, 0);
    request_entries(nxt, 1);
    if constexpr (KVR) {
        request_first_row_numbers(cur, 0);
        request_first_row_numbers(nxt, 1);
        VMOBA_WAIT_VMCNT(0);
        __syncthreads();
    }
    begin_k(cur);
    begin_v(cur);
    static_for<4>([&](auto x) {
        constexpr int X = decltype(x)::value;
        if constexpr (KVR && X < 2) vrow = row_number(X, 0);
        if (X == 1 && cur.L <= G) zero_v();
        if constexpr (KVR) {
            dma_row16<X * SLOT>(k_base, row_number(X, 0), kss, pc16, lds_rows);
            if constexpr (X < 2) dma_row16<V0 + X * SLOT>(v_base, vrow, vss, pc16, lds_rows);
        } else {
            dma16_advance(k_base, min(k_off, k_last), k_off, k_adv, lds_rows, X * SLOT);
            if constexpr (X < 2) dma16_advance(v_base, min(v_off, v_last), v_off, v_adv, lds_rows, V0 + X * SLOT);
        }
    });
    VMOBA_WAIT_VMCNT(6);                   // the list entries are here
    request_queries(cur, 0);
    VMOBA_WAIT_VMCNT(0);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) read_query(ks);
    f32x16_t oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt] = zero16;
    float m_run = 0.f, l_run = 0.f, limit = 0.f, m_out = 0.f, l_out = 0.f;      // l: this lane half's share of the row sum; _out: of the tile before
    bf16x8_t opK[4], opV[4];                    // operands of units u .. u + 2, slot = unit % 4
    f32x16_t sA = zero16, sB = zero16;
    const bf16x8_t p_none = __builtin_bit_cast(bf16x8_t, u32x4_t{0u, 0u, 0u, 0u});
    bf16x8_t pA[2] = {p_none, p_none}, pB[2] = {p_none, p_none};
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(readK(0, ks), qf[ks], sA, 0, 0, 0);
    opK[0] = readK(SLOT, 0);
    opK[1] = readK(SLOT, 1);
    opV[0] = opK[0];                            // (the first step's second product is thrown away)
    opV[1] = opK[1];
    int g = 0, Ge = groups_of(cur);             // group of `cur` and the number of them
    if constexpr (KVR) {
        krow = Ge > 4 ? row_number(4, 0) : row_number(0, 1);
        vrow = row_number(2, 0);
    }

    bool surplus = false;                       // SHORT: the last group of the tile before has no key
    enum { FIRST, SECOND, THIRD, MIDDLE, BEFORE_LAST, LAST };
    // One step; which of the tile's it is, is compile-time.
    auto step = [&](auto which, f32x16_t& s_cur, f32x16_t& s_nxt, bf16x8_t(&p_new)[2], bf16x8_t(&p_prev)[2]) __attribute__((always_inline)) {
        constexpr int WHICH = decltype(which)::value;
        // SHORT: what the step's three groups g + 1, g and g - 1 have to do
        constexpr bool ENDS = SHORT && WHICH != THIRD && WHICH != MIDDLE;
        const bool qk = !ENDS || WHICH == LAST || (g + 1) * G < cur.L, sm = !ENDS || WHICH == FIRST || g * G < cur.L,
                   pv = !ENDS || (WHICH == FIRST ? !surplus : (g - 1) * G < cur.L);
        if constexpr (WHICH == SECOND || WHICH == THIRD) VMOBA_WAIT_VMCNT(N_STEP + N_FIRST);       // the first step's rows are older than its other requests
        else VMOBA_WAIT_VMCNT(N_STEP);
        asm volatile("s_barrier" ::: "memory");
        if constexpr (WHICH != THIRD && WHICH != MIDDLE) {
            if (sm && __builtin_expect((g + 1) * G > cur.L, WHICH == LAST)) {     // keys past the block's end; accumulator value i is key row acc_row(i, 0) + hf
                const int vh = cur.L - g * G - hf;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (acc_row(i, 0) >= vh) s_cur[i] = -INFINITY;
            }
        }
        float alpha = 1.f;
        int raised = 0;                         // (opaque: otherwise the comparison is kept instead)
        asm volatile("" : "+s"(raised));
        uint32_t w[8];                          // P of this step as packed bf16 pairs (accumulator values 2j, 2j + 1)
        if constexpr (ENDS && WHICH != FIRST)
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = 0u;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int u2 = u + 2;
            const bf16x8_t nk = u2 < UNITS ? readK(r1, u2) : readK(r2, u2 - UNITS);
            const bf16x8_t nv = u2 < UNITS ? readV(r3, u2) : readV(r0, u2 - UNITS);
            if (qk) s_nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opK[u & 3], qf[u], u == 0 ? zero16 : s_nxt, 0, 0, 0);
            // (the tile's second step begins its second product)
            if (pv) oacc[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opV[u & 3], p_prev[u / DT], WHICH == SECOND && u < DT ? zero16 : oacc[u % DT], 0, 0, 0);
            if constexpr (WHICH == BEFORE_LAST) read_query(u);      // the next step's first product is the next tile's first
            if (sm && u == 0) {
                float mx = fmaxf(s_cur[0], s_cur[1]);
#pragma unroll
                for (int i = 2; i < 16; i += 2) mx = fmaxf(fmaxf(mx, s_cur[i]), s_cur[i + 1]);
                if constexpr (WHICH == FIRST) {
                    m_out = m_run;
                    l_out = l_run;
                    mx = swap_halves_max(mx);
                    m_run = mx * scale_log2;                         // scale_log2 > 0
                    limit = mx + lazy;
                    l_run = 0.f;
                } else if (__builtin_expect(__builtin_amdgcn_ballot_w64(mx > limit) != 0, 0)) {      // some row's new maximum passes its limit
                    asm volatile("" : "+v"(mx));
                    mx = swap_halves_max(mx);
                    const float m_new = mx > limit ? mx * scale_log2 : m_run;
                    alpha = exp2_raw(m_run - m_new);
                    limit = mx > limit ? mx + lazy : limit;
                    m_run = m_new;
                    l_run *= alpha;
                    raised = 1;
                }
            }
            // 8 value pairs over the other units; a pair is packed as soon as it exists
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (sm && 1 + j * (UNITS - 1) / 8 == u) {
                    const float p0 = exp2_raw(fmaf(s_cur[2 * j], scale_log2, -m_run));
                    const float p1 = exp2_raw(fmaf(s_cur[2 * j + 1], scale_log2, -m_run));
                    l_run += p0 + p1;
                    w[j] = pack_bf16x2(p0, p1);
                    asm volatile("" : "+v"(w[j]));  // keeps the pair in this unit (it is only read a step later)
                }
            }
            asm volatile("" : "+v"(l_run));
            if (u == 1) {
                // K(n+4) into the slot of K(n), V(n+2) into that of V(n-2)
                if constexpr (WHICH < BEFORE_LAST) {
                    if (__builtin_expect(g == Ge - 4, 0)) begin_k(nxt);
                } else if constexpr (WHICH == BEFORE_LAST) {
                    begin_v(nxt);
                }
                if constexpr (WHICH == FIRST || WHICH == SECOND) {
                    if (__builtin_expect((g + 2) * G >= cur.L, 0)) zero_v();
                } else if constexpr (WHICH == LAST) {
                    if (__builtin_expect(nxt.L <= G, 0)) zero_v();
                }
                if constexpr (KVR) {
                    const int tn = ring_ahead(1);
                    dma_row16<0>(k_base, krow, kss, pc16, lds_rows + r0);
                    dma_row16<V0>(v_base, vrow, vss, pc16, lds_rows + r2);
                    // for the next step (after the last one: group 4 of the next tile or, if that has no more than four, the first of the one behind it)
                    if (WHICH == LAST && groups_of(nxt) == 4) krow = row_number(0, ring_ahead(2));
                    else krow = g + 5 < Ge ? row_number(g + 5, tp) : row_number(g + 5 - Ge, tn);
                    vrow = g + 3 < Ge ? row_number(g + 3, tp) : row_number(g + 3 - Ge, tn);
                    // every wavefront by itself: its row numbers then need no barrier and all waits the same count
                    request_row_numbers(cur, g + 8, tp);
                } else {
                    dma16_advance(k_base, min(k_off, k_last), k_off, k_adv, lds_rows, r0);
                    dma16_advance(v_base, min(v_off, v_last), v_off, v_adv, lds_rows + V0, r2);
                }
            }
            opK[u2 & 3] = nk;
            opV[u2 & 3] = nv;
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (WHICH != FIRST) {
            if (__builtin_expect(raised, 0)) {  // the accumulator holds groups <= g - 1, all relative to the old maximum
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[dt][i] *= alpha;
            }
        }
        const u32x4_t lo = {w[0], w[1], w[2], w[3]}, hi = {w[4], w[5], w[6], w[7]};
        p_new[0] = __builtin_bit_cast(bf16x8_t, lo);
        p_new[1] = __builtin_bit_cast(bf16x8_t, hi);
        const uint32_t r = r0;
        r0 = r1;
        r1 = r2;
        r2 = r3;
        r3 = r;
        ++g;
    };
    // Partial rows of the tile before: O^T value i of tile dt <-> channel 32*dt + 8*(i>>2) + 4*hf + (i&3)
    auto write_partials = [&]() {
        const float l_tot = swap_halves_sum(l_out);
        const float inv = 1.f / l_tot;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                u32x2_t v;
                v.x = pack_bf16x2(oacc[dt][4 * gq + 0] * inv, oacc[dt][4 * gq + 1] * inv);
                v.y = pack_bf16x2(oacc[dt][4 * gq + 2] * inv, oacc[dt][4 * gq + 3] * inv);
                *reinterpret_cast<u32x2_t*>(mine + l32 * OPITCH + (dt * 32 + gq * 8 + hf * 4) * 2) = v;
            }
        // the tile's partials are consecutive rows of Opart (bfloat16): row = first pair of the tile + entry
        const auto a = args();
        constexpr int LPR = D * 2 / 16;                                       // lanes per row
        char* dst = reinterpret_cast<char*>(a->Opart) + out_pair * (D * 2) + lane % LPR * 16;
        const int row0 = wave * 32 + lane / LPR;
        u32x4_t x[32 * LPR / 64];
#pragma unroll
        for (int k = 0; k < 32 * LPR / 64; ++k) x[k] = *reinterpret_cast<const u32x4_t*>(mine + (k * (64 / LPR) + lane / LPR) * OPITCH + lane % LPR * 16);
        if (__builtin_expect(wave * 32 + 31 <= out_last, 1)) {
#pragma unroll
            for (int k = 0; k < 32 * LPR / 64; ++k) *reinterpret_cast<u32x4_t*>(dst + (row0 + k * (64 / LPR)) * (D * 2)) = x[k];
        } else {
#pragma unroll
            for (int k = 0; k < 32 * LPR / 64; ++k) *reinterpret_cast<u32x4_t*>(dst + min(row0 + k * (64 / LPR), out_last) * (D * 2)) = x[k];
        }
        a->lse_part[out_pair + min(wave * 32 + l32, out_last)] = (m_out + log2f(l_tot)) * LN2;
    };
    using First = std::integral_constant<int, FIRST>;
    using Second = std::integral_constant<int, SECOND>;
    using Third = std::integral_constant<int, THIRD>;
    using Middle = std::integral_constant<int, MIDDLE>;
    using BeforeLast = std::integral_constant<int, BEFORE_LAST>;
    using Last = std::integral_constant<int, LAST>;
    for (;;) {
        step(First{}, sA, sB, pB, pA);
        if constexpr (KVR) request_first_row_numbers(nn, ring_ahead(2));
        if (__builtin_expect(out_last >= 0, 1)) write_partials();
        request_descriptor(f_next);
        request_entries(nn, par);
        request_queries(nxt, par ^ 1);
        if (__builtin_expect(out_last < 0, 0)) VMOBA_WAIT_VMCNT(0);          // (no partial rows: the waits would count too few)
        step(Second{}, sB, sA, pA, pB);
        if (Ge > 4) {
            step(Third{}, sA, sB, pB, pA);
            while (g < Ge - 3) {                // the steps come in pairs that swap the two register sets
                step(Middle{}, sB, sA, pA, pB);
                step(Middle{}, sA, sB, pB, pA);
            }
            if (g < Ge - 2) {
                step(Middle{}, sB, sA, pA, pB);
            } else {
                sA = sB;
                pA[0] = pB[0];
                pA[1] = pB[1];
            }
        }
        step(BeforeLast{}, sA, sB, pB, pA);
        step(Last{}, sB, sA, pA, pB);
        if constexpr (SHORT) surplus = (Ge - 1) * G >= cur.L;
        out_pair = cur.pair;
        out_last = cur.count - 1;
        // (SHORT leaves at the loop's end: from here the compiler copies registers whose values nothing uses, and in that form it does so right
        // behind matrix instructions that may still be writing them)
        if (!SHORT && --tiles_left == 0) break;
        const u32x4_t d = *reinterpret_cast<const u32x4_t*>(smem + DESC0 + wave * 256);
        cur = nxt;
        nxt = nn;
        nn = make_tile(make_int4(__builtin_amdgcn_readfirstlane((int)d.x), __builtin_amdgcn_readfirstlane((int)d.y),
                                 __builtin_amdgcn_readfirstlane((int)d.z), __builtin_amdgcn_readfirstlane((int)d.w)), nxt);
        f_next += f_step;
        g = 0;
        Ge = groups_of(cur);
        par ^= 1;
        tp = ring_ahead(1);
        if (SHORT && --tiles_left == 0) break;
    }
    // second product of the last tile's last group
    VMOBA_WAIT_VMCNT(0);                   // (no request may reach LDS that belongs to another workgroup by the kernel's end, either)
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int u = 0; u < UNITS; ++u) oacc[u % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(readV(r3, u), pA[u / DT], oacc[u % DT], 0, 0, 0);
    m_out = m_run;
    l_out = l_run;
    write_partials();
}

// ---------------------------------------------------------------------------------------------
// Merge: O[q] = sum_pairs exp(lse_pair - LSE[q]) * Opart[pair], LSE[q] = logsumexp(lse_pair).
// A group of lanes per query, each owning CH consecutive channels (one 16-byte load per partial).
// Partials have the tensors' type.
// A head whose selection did not fit the lists (row_ptr[S] > cap, see vmoba_select) counts as having selected nothing.
template <bool BF16, int D>
__global__ __launch_bounds__(256) void attn_fwd_merge_kernel(const float* __restrict__ Opart, const float* __restrict__ lse_part,
                                                             const int* __restrict__ row_ptr, const int* __restrict__ pair_pos,
                                                             TensorView O, float* __restrict__ LSE,
                                                             const int* __restrict__ out_rows, int Hh, int S, long long cap) {
    constexpr int CH = BF16 ? 8 : 4;
    constexpr int MB = 8;                    // partial rows in flight per lane
    constexpr int LPQ = D / CH;              // lanes per query
    constexpr int QPW = 256 / LPQ;           // queries per workgroup
    const int bh = blockIdx.y, b = bh / Hh, h = bh % Hh;
    const int q = blockIdx.x * QPW + threadIdx.x / LPQ;
    const int part = threadIdx.x % LPQ;
    if (q >= S) return;
    const bool fits = row_ptr[(long long)bh * (S + 1) + S] <= cap;
    const int r0 = row_ptr[(long long)bh * (S + 1) + q];
    const int r1 = fits ? row_ptr[(long long)bh * (S + 1) + q + 1] : r0;
    const long long seg = (long long)bh * cap;
    // one pass with a running maximum; MB partials in flight per step (index -> lse and row loads)
    float mx = -INFINITY;
    float acc[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[c] = 0.f;
    float wsum = 0.f;
    for (int r = r0; r < r1; r += MB) {
        long long pair[MB];
        float l[MB];
#pragma unroll
        for (int u = 0; u < MB; ++u) pair[u] = seg + pair_pos[seg + min(r + u, r1 - 1)];
#pragma unroll
        for (int u = 0; u < MB; ++u) l[u] = (r + u < r1) ? lse_part[pair[u]] : -INFINITY;
        float v[MB][CH];
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            if constexpr (BF16) {
                // (read once: a non-temporal load, so the rows do not displace what the L2 holds; -7 % kernel time)
                const u32x4_t x = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(Opart) + pair[u] * D + part * 8));
                v[u][0] = bf16lo_to_f32(x.x); v[u][1] = bf16hi_to_f32(x.x); v[u][2] = bf16lo_to_f32(x.y); v[u][3] = bf16hi_to_f32(x.y);
                v[u][4] = bf16lo_to_f32(x.z); v[u][5] = bf16hi_to_f32(x.z); v[u][6] = bf16lo_to_f32(x.w); v[u][7] = bf16hi_to_f32(x.w);
            } else {
                const f32x4_t x = *reinterpret_cast<const f32x4_t*>(Opart + pair[u] * D + part * 4);
                v[u][0] = x.x; v[u][1] = x.y; v[u][2] = x.z; v[u][3] = x.w;
            }
        }
        float m_new = mx;
#pragma unroll
        for (int u = 0; u < MB; ++u) m_new = fmaxf(m_new, l[u]);
        const float alpha = expf(mx - m_new);          // exp(-inf) = 0 on the first step (m_new is finite: l[0] is)
        wsum *= alpha;
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[c] *= alpha;
#pragma unroll
        for (int u = 0; u < MB; ++u) {
            const float w = expf(l[u] - m_new);        // 0 for the padding entries
            wsum += w;
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[c] += w * v[u][c];
        }
        mx = m_new;
    }
    float lse = -INFINITY;
    if (r1 > r0) {
        const float inv = 1.f / wsum;
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[c] *= inv;
        lse = mx + logf(wsum);
    }
    const int qo = out_rows ? out_rows[q] : q;       // row of O that block-order row q is written to
    char* dst = O.ptr + ((long long)b * O.stride_b + (long long)qo * O.stride_s + (long long)h * O.stride_h) * (BF16 ? 2 : 4);
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
    if (part == 0) LSE[(long long)bh * S + q] = lse;
}

struct FwdWs {
    float* Opart;      // [BH * cap][D], in the tensors' type
    float* lse_part;   // [BH * cap]
    int4* tile_desc;   // the flat list of all heads' tiles
    int* n_tiles;      // its length, then the split kernels' flag
    int* head_tiles;   // [BH]
    char* Q3;          // split kernels: [BH][S][3][D], the terms of Q, and [BH][S][6][D], those of K and V in block order (see attn_split.hip)
    char* KV6;
    size_t total;
};

}  // namespace

void launch_head_tiles(hipStream_t st, const int* blk_ptr, int* head_tiles, int BH, int nb, int TM) {
    head_tiles_kernel<<<dim3((unsigned)ceil_div64(BH, 4)), dim3(256), 0, st>>>(blk_ptr, head_tiles, BH, nb, TM);
}
// Grid width (tiles per head) for tiles of TM list entries: a host-side bound on sum_j ceil(cnt_j / TM).
int64_t vmoba_max_tiles(int64_t cap, int TM) { return (cap / TM + VMOBA_MAX_BLOCKS + 7) / 8 * 8; }
namespace {

FwdWs carve_fwd(void* base, int BH, int64_t S, int D, int64_t cap, int es, bool split) {       // es: bytes per element of the partial rows
    FwdWs w;
    char* p = (char*)base;
    size_t off = 0;
    w.Opart = (float*)(p + off);     off += align_up((size_t)BH * cap * D * es, 256);
    w.lse_part = (float*)(p + off);  off += align_up((size_t)BH * cap * 4, 256);
    w.tile_desc = (int4*)(p + off);  off += align_up((size_t)BH * vmoba_max_tiles(cap, 64) * 16, 256);
    w.n_tiles = (int*)(p + off);     off += 256;
    w.head_tiles = (int*)(p + off);  off += align_up((size_t)BH * 4, 256);
    w.Q3 = p + off;                  off += split ? align_up((size_t)BH * S * 6 * D, 256) : 0;
    w.KV6 = p + off;                 off += split ? align_up((size_t)BH * S * 12 * D, 256) : 0;
    w.total = off;
    return w;
}

}  // namespace

size_t vmoba_attn_fwd_workspace_bytes(int B, int Hh, int64_t S, int D, int nb, int64_t cap, int dtype) {
    const bool bf16 = dtype == VMOBA_BF16;
    return carve_fwd(nullptr, B * Hh, S, D, cap, bf16 ? 2 : 4, !bf16 && use_split(B * Hh, S, D, nb, cap)).total;
}

// Compute units of the current device (queried once).
int vmoba_num_cus() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            n = v;
        else
            n = 256;
    }
    return n;
}

extern "C" int vmoba_attn_fwd(int B, int Hh, int64_t S, int D, int32_t n_blocks, const int32_t* blk_off,
                              const vmoba_tensor* Qp, const vmoba_tensor* Kp, const vmoba_tensor* Vp,
                              const int32_t* blk_ptr, const int32_t* q_idx, const int32_t* row_ptr,
                              const int32_t* pair_pos, int64_t nnz_capacity, float softmax_scale,
                              const vmoba_tensor* O, float* LSE, const int32_t* out_rows, const int32_t* kv_rows,
                              void* workspace, size_t workspace_bytes, void* stream) {
    if (B <= 0 || Hh <= 0 || S <= 0 || n_blocks <= 0 || nnz_capacity <= 0) return VMOBA_ERR_INVALID_ARG;
    if (!blk_off || !blk_ptr || !q_idx || !row_ptr || !pair_pos || !LSE || !workspace) return VMOBA_ERR_INVALID_ARG;
    if (!tensor_ok(Qp) || !tensor_ok(Kp) || !tensor_ok(Vp) || !tensor_ok(O)) return VMOBA_ERR_INVALID_ARG;
    if (!std::isfinite(softmax_scale)) return VMOBA_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return VMOBA_ERR_UNSUPPORTED;
    if (n_blocks > VMOBA_MAX_BLOCKS) return VMOBA_ERR_UNSUPPORTED;
    const int dt = Qp->dtype;
    if (Kp->dtype != dt || Vp->dtype != dt || O->dtype != dt) return VMOBA_ERR_UNSUPPORTED;
    const int BH = B * Hh;
    if (nnz_capacity > INT32_MAX || (int64_t)BH * nnz_capacity * D > ((int64_t)1 << 40)) return VMOBA_ERR_UNSUPPORTED;
    const bool bf16 = dt == VMOBA_BF16;
    const bool split = !bf16 && use_split(BH, S, D, n_blocks, nnz_capacity);
    FwdWs ws = carve_fwd(workspace, BH, S, D, nnz_capacity, bf16 ? 2 : 4, split);
    if (workspace_bytes < ws.total) return VMOBA_ERR_WORKSPACE;
    if (((uintptr_t)workspace) & 255) return VMOBA_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    const TensorView Qv = make_view(Qp), Kv = make_view(Kp), Vv = make_view(Vp), Ov = make_view(O);
    const float scale_log2 = softmax_scale * LOG2E;
    // the bfloat16 kernel addresses the rows of one (batch, head) slice of K and V with 32-bit byte offsets
    if (bf16 && (Kp->stride_s <= 0 || Vp->stride_s <= 0 ||
                 (uint64_t)(S + 256) * (uint64_t)Kp->stride_s * 2 >= ((uint64_t)1 << 32) ||
                 (uint64_t)(S + 256) * (uint64_t)Vp->stride_s * 2 >= ((uint64_t)1 << 32)))
        return VMOBA_ERR_UNSUPPORTED;
    // with keys in place a row's byte offset is one 24-bit multiply of its row number and the row stride
    if (bf16 && kv_rows && (S >= (1 << 24) || Kp->stride_s * 2 >= (1 << 24) || Vp->stride_s * 2 >= (1 << 24)))
        return VMOBA_ERR_UNSUPPORTED;
    // bf16, D = 128: 256-query tiles, one persistent workgroup of 8 wavefronts per compute unit (a tile's K and V
    // rows are fetched once per 256 queries); D = 64: 128-query tiles, two workgroups of 4 wavefronts per compute unit;
    // float32: one workgroup per tile of 128 queries
    const bool wide = bf16 && D == 128;
    const int TM = wide ? 256 : 128;
    const int64_t max_tiles = std::min<int64_t>(vmoba_max_tiles(nnz_capacity, TM), (nnz_capacity / TM + n_blocks + 7) / 8 * 8);
    const int* head_tiles = heads_counted_first(BH, n_blocks) ? ws.head_tiles : nullptr;
    if (head_tiles) launch_head_tiles(st, blk_ptr, ws.head_tiles, BH, n_blocks, TM);
    tile_list_kernel<<<dim3((unsigned)ceil_div64(max_tiles, 256), (unsigned)BH), dim3(256), 0, st>>>(
        blk_ptr, blk_off, head_tiles, ws.tile_desc, ws.n_tiles, split ? ws.n_tiles + 1 : nullptr, BH, n_blocks, TM);
    VMOBA_CHECK_LAUNCH();
    if (split) {
        launch_split_rows(D, BH, Hh, (int)S, st, Qv, nullptr, ws.Q3, 3, 0, ws.n_tiles + 1);
        launch_split_rows(D, BH, Hh, (int)S, st, Kv, kv_rows, ws.KV6, 6, 0, ws.n_tiles + 1);
        launch_split_rows(D, BH, Hh, (int)S, st, Vv, kv_rows, ws.KV6, 6, 3, ws.n_tiles + 1);
        VMOBA_CHECK_LAUNCH();
    }
    VMOBA_PROFILE_BEGIN(0, st);
    if (!bf16) {
        const dim3 grid = flat_tile_grid(BH, max_tiles, nnz_capacity, TM, n_blocks);
        if (split)
            launch_fwd_tiles_split(D, grid, st, ws.Q3, ws.KV6, q_idx, ws.tile_desc, ws.n_tiles, ws.n_tiles + 1, ws.Opart, ws.lse_part, (int)S,
                                   (long long)nnz_capacity, scale_log2);
        launch_fwd_tiles_f32(D, grid, st, split ? ws.n_tiles + 1 : nullptr, Qv, Kv, Vv, q_idx, ws.tile_desc, ws.n_tiles,
                             ws.Opart, ws.lse_part, Hh, (long long)nnz_capacity, scale_log2, kv_rows);
    } else {
        // the kernel's running maximum and its mask of the keys past a block's end need a positive scale: the sign goes to Q, and the
        // smallest normal number does for 0 (it leaves every weight at 1)
        const float magnitude = std::max(std::fabs(scale_log2), FLT_MIN);
        const int q_offsets_32 = S < (1 << 24) && Qp->stride_s > 0 && Qp->stride_s * 2 < (1 << 24) && (uint64_t)S * (uint64_t)Qp->stride_s * 2 < ((uint64_t)1 << 32);
        const dim3 pgrid((unsigned)std::min<int64_t>((wide ? 1 : 2) * (int64_t)vmoba_num_cus(), (int64_t)BH * max_tiles));
#define MFMA_ARGS FwdArgs{Qv, Kv, Vv, q_idx, ws.tile_desc, ws.n_tiles, ws.Opart, ws.lse_part, (long long)nnz_capacity, kv_rows, Hh, magnitude, q_offsets_32}
#define LAUNCH_FWD(NEG, SHORT)                                                                                                \
    do {                                                                                                                      \
        if (wide && kv_rows) attn_fwd_tile_mfma_kernel<128, 8, true, NEG, SHORT><<<pgrid, dim3(512), 0, st>>>(MFMA_ARGS);     \
        else if (wide) attn_fwd_tile_mfma_kernel<128, 8, false, NEG, SHORT><<<pgrid, dim3(512), 0, st>>>(MFMA_ARGS);          \
        else if (kv_rows) attn_fwd_tile_mfma_kernel<64, 4, true, NEG, SHORT><<<pgrid, dim3(256), 0, st>>>(MFMA_ARGS);         \
        else attn_fwd_tile_mfma_kernel<64, 4, false, NEG, SHORT><<<pgrid, dim3(256), 0, st>>>(MFMA_ARGS);                     \
    } while (0)
        if (scale_log2 < 0.f) LAUNCH_FWD(true, false);
        else if (S / n_blocks <= SHORT_BLOCK) LAUNCH_FWD(false, true);
        else LAUNCH_FWD(false, false);
#undef LAUNCH_FWD
#undef MFMA_ARGS
    }
    VMOBA_PROFILE_END(0, st);
    VMOBA_CHECK_LAUNCH();
    const int qpw = 256 / (D / (bf16 ? 8 : 4));     // partials in the tensors' type
    dim3 mgrid((unsigned)ceil_div64(S, qpw), (unsigned)BH);
#define MERGE_ARGS ws.Opart, ws.lse_part, row_ptr, pair_pos, Ov, LSE, out_rows, Hh, (int)S, (long long)nnz_capacity
    if (bf16 && D == 128) attn_fwd_merge_kernel<true, 128><<<mgrid, dim3(256), 0, st>>>(MERGE_ARGS);
    else if (bf16) attn_fwd_merge_kernel<true, 64><<<mgrid, dim3(256), 0, st>>>(MERGE_ARGS);
    else if (D == 128) attn_fwd_merge_kernel<false, 128><<<mgrid, dim3(256), 0, st>>>(MERGE_ARGS);
    else attn_fwd_merge_kernel<false, 64><<<mgrid, dim3(256), 0, st>>>(MERGE_ARGS);
#undef MERGE_ARGS
    VMOBA_CHECK_LAUNCH();
    return VMOBA_OK;
}
