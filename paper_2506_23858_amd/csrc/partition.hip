// vmoba_partition: token -> key-block rearrangement of Sec. 3.2, Eq. 1 (and its inverse).
// One kernel: a workgroup takes a run of 16-byte pieces of the (token, head) rows in block order, finds the tokens of its positions -- from the grid
// description in closed form (and then also writes its part of perm / inv_perm / blk_off), or from
// perm -- and moves 16-byte pieces of the (token, head) rows between the caller's order and block
// order.  (With the index arrays in a launch of their own a small call spent a third of its time there.)
#include "common.h"
#include <algorithm>

namespace {

struct GridDesc {
    int T, H, W, bt, bh, bw;
    long long chunk;
    int nH, nW;
    int S, n_blocks;
};

// Block-order position -> token (row-major index of the grid), block and rank inside the block.
struct Place { int token, block, rank; };
__device__ __forceinline__ Place place_of(const GridDesc& g, int p) {
    Place r;
    if (g.chunk > 0) {
        r.token = p;
        r.block = (int)(p / g.chunk);
        r.rank = (int)(p - (long long)r.block * g.chunk);
        return r;
    }
    // positions count the slabs along T, inside a slab the strips along H, inside a strip the boxes along W; only the
    // last of each can be thinner than the rest
    const int it = p / (g.bt * g.H * g.W), t0 = it * g.bt, et = min(g.bt, g.T - t0);
    p -= t0 * g.H * g.W;
    const int ih = p / (et * g.bh * g.W), h0 = ih * g.bh, eh = min(g.bh, g.H - h0);
    p -= et * h0 * g.W;
    const int iw = p / (et * eh * g.bw), w0 = iw * g.bw, ew = min(g.bw, g.W - w0);
    p -= et * eh * w0;
    const int t = p / (eh * ew), q = p - t * (eh * ew), h = q / ew, w = q - h * ew;
    r.token = ((t0 + t) * g.H + h0 + h) * g.W + w0 + w;
    r.block = (it * g.nH + ih) * g.nW + iw;
    r.rank = p;
    return r;
}

struct CopyDesc {
    TensorView in[8], out[8];
    int in_bf16[8], out_bf16[8];
    int n_tensors;
};

// The 16-byte pieces of one batch element's INPUT rows are numbered (position, head, piece), the piece fastest, so a wavefront reads
// whole rows and, in the caller's layout, the heads of one token that lie next to each other; a workgroup moves
// CHUNK consecutive ones.
// BUILD: perm, inv_perm and blk_off are written (by the workgroups of the first batch element and tensor, every position by the one that
// holds its first piece) instead of perm being read.
// Bound by HBM (5.2 to 6.7 TB/s).  What matters is how much a workgroup moves: with gathered reads 256 pieces, one per thread, with scattered
// writes 512.  Q, K, V of 40 heads x 32 760 tokens with 2048 / 1024 / 512 / 256 pieces: 391 / 377 / 374 / 336 us, K and V of 12 heads
// x 112 320 tokens 261 / 253 / 260 / 235; the inverse of one tensor, 40 heads, 131 / 123 / 123 / 133.
constexpr int chunk_pieces(bool inverse) { return inverse ? 512 : 256; }
constexpr int INDEX_CHUNK = 256;                       // positions per workgroup when only the index arrays are wanted
template <bool INVERSE, bool BUILD>
__global__ __launch_bounds__(256) void permute_rows_kernel(GridDesc g, CopyDesc d, int* __restrict__ perm, int* __restrict__ inv_perm,
                                                           int* __restrict__ blk_off, int Hh, int D, unsigned chunk0) {
    constexpr int CHUNK = chunk_pieces(INVERSE), U = CHUNK / 256;
    __shared__ int sTok[INDEX_CHUNK];
    static_assert(CHUNK / 8 + 1 <= INDEX_CHUNK && INDEX_CHUNK <= 256, "a thread per position of the workgroup");
    const int t = blockIdx.z, b = blockIdx.y, tid = threadIdx.x;
    const bool copy = t < d.n_tensors;
    const int in_es = d.in_bf16[t] ? 2 : 4;
    const int sh = __builtin_ctz(D * in_es / 16);      // 8, 16 or 32 pieces per input row
    const unsigned per_pos = copy ? (unsigned)Hh << sh : 1u, chunk = copy ? CHUNK : INDEX_CHUNK;
    const unsigned long long total = (unsigned long long)g.S * per_pos, first = ((unsigned long long)chunk0 + blockIdx.x) * chunk;
    if (first >= total) return;
    const int p0 = (int)(total >> 32 ? first / per_pos : (unsigned)first / per_pos);
    const int skip = (int)(first - (unsigned long long)p0 * per_pos);       // pieces of position p0 that belong to the workgroup before
    const int np = min((int)((skip + chunk - 1) / per_pos) + 1, g.S - p0);
    if (tid < np) {
        const int p = p0 + tid;
        if constexpr (BUILD) {
            const Place pl = place_of(g, p);
            sTok[tid] = pl.token;
            if (b == 0 && t == 0 && (tid > 0 || skip == 0)) {
                perm[p] = pl.token;
                inv_perm[pl.token] = p;
                if (pl.rank == 0) blk_off[pl.block] = p;
                if (p == 0) blk_off[g.n_blocks] = g.S;
            }
        } else {
            sTok[tid] = perm[p];
        }
    }
    if (!copy) return;                                 // only the index arrays are wanted
    __syncthreads();
    const TensorView in = d.in[t], out = d.out[t];
    const bool cvt = (!d.in_bf16[t]) && d.out_bf16[t];
    const char* in_b = in.ptr + (long long)b * in.stride_b * in_es;
    char* out_b = out.ptr + (long long)b * out.stride_b * (cvt ? 2 : in_es);
    const float inv_hh = 1.f / (float)Hh;
    const int n_items = (int)min((unsigned long long)CHUNK, total - first);
    u32x4_t v[U];
    char* dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = skip + min(tid + 256 * u, n_items - 1);
        const int piece = i & ((1 << sh) - 1), r = i >> sh;
        int pl = (int)((float)r * inv_hh);             // r / Hh, one off at most
        if (pl * Hh > r) --pl;
        if ((pl + 1) * Hh <= r) ++pl;
        const int h = r - pl * Hh;
        const int tok = sTok[pl], s_in = INVERSE ? p0 + pl : tok, s_out = INVERSE ? tok : p0 + pl;
        v[u] = *reinterpret_cast<const u32x4_t*>(in_b + ((long long)s_in * in.stride_s + (long long)h * in.stride_h) * in_es + piece * 16);
        dst[u] = out_b + ((long long)s_out * out.stride_s + (long long)h * out.stride_h) * (cvt ? 2 : in_es) + piece * (cvt ? 8 : 16);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (tid + 256 * u >= n_items) break;
        if (!cvt) {
            *reinterpret_cast<u32x4_t*>(dst[u]) = v[u];
        } else {
            u32x2_t w;
            w.x = pack_bf16x2(__uint_as_float(v[u].x), __uint_as_float(v[u].y));
            w.y = pack_bf16x2(__uint_as_float(v[u].z), __uint_as_float(v[u].w));
            *reinterpret_cast<u32x2_t*>(dst[u]) = w;
        }
    }
}

bool grid_ok(const vmoba_grid* g) {
    if (!g) return false;
    if (g->T <= 0 || g->H <= 0 || g->W <= 0) return false;
    if ((int64_t)g->T * g->H * g->W > (int64_t)1 << 30) return false;
    if (g->chunk > 0) return true;
    if (g->chunk < 0) return false;
    return g->bt > 0 && g->bh > 0 && g->bw > 0;
}

}  // namespace

extern "C" int vmoba_layer_kind(int layer) { return ((layer % 3) + 3) % 3; }

extern "C" int vmoba_partition_dims(const vmoba_grid* g, int64_t* S, int32_t* n_blocks) {
    if (!grid_ok(g) || !S || !n_blocks) return VMOBA_ERR_INVALID_ARG;
    int64_t s = (int64_t)g->T * g->H * g->W;
    int64_t nb;
    if (g->chunk > 0) {
        nb = ceil_div64(s, g->chunk);
    } else {
        nb = ceil_div64(g->T, g->bt) * ceil_div64(g->H, g->bh) * ceil_div64(g->W, g->bw);
    }
    if (nb > INT32_MAX) return VMOBA_ERR_UNSUPPORTED;
    *S = s;
    *n_blocks = (int32_t)nb;
    return VMOBA_OK;
}

extern "C" int vmoba_partition(const vmoba_grid* g, int inverse, int B, int Hh, int D, int n_tensors,
                               const vmoba_tensor* in, const vmoba_tensor* out, int32_t* perm,
                               int32_t* inv_perm, int32_t* blk_off, void* stream) {
    int64_t S;
    int32_t nb;
    int rc = vmoba_partition_dims(g, &S, &nb);
    if (rc != VMOBA_OK) return rc;
    if (B <= 0 || Hh <= 0 || n_tensors < 0 || n_tensors > 8) return VMOBA_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return VMOBA_ERR_UNSUPPORTED;
    if (!perm) return VMOBA_ERR_INVALID_ARG;
    const bool build_index = !inverse && (inv_perm || blk_off);   // both null: perm is reused as given
    if (build_index && (!inv_perm || !blk_off)) return VMOBA_ERR_INVALID_ARG;
    if (n_tensors > 0 && (!in || !out)) return VMOBA_ERR_INVALID_ARG;
    CopyDesc cd = {};
    cd.n_tensors = n_tensors;
    for (int i = 0; i < n_tensors; ++i) {
        if (!tensor_ok(&in[i]) || !tensor_ok(&out[i])) return VMOBA_ERR_INVALID_ARG;
        bool same = in[i].dtype == out[i].dtype;
        bool down = in[i].dtype == VMOBA_F32 && out[i].dtype == VMOBA_BF16;
        if (!same && !down) return VMOBA_ERR_UNSUPPORTED;
        cd.in[i] = make_view(&in[i]);
        cd.out[i] = make_view(&out[i]);
        cd.in_bf16[i] = in[i].dtype == VMOBA_BF16;
        cd.out_bf16[i] = out[i].dtype == VMOBA_BF16;
    }
    if (!build_index && n_tensors == 0) return VMOBA_OK;
    hipStream_t st = (hipStream_t)stream;
    GridDesc gd;
    gd.T = g->T; gd.H = g->H; gd.W = g->W;
    gd.bt = g->bt; gd.bh = g->bh; gd.bw = g->bw;
    gd.chunk = g->chunk;
    if (g->chunk > 0) {
        gd.nH = gd.nW = 1;
        gd.bt = gd.bh = gd.bw = 1;
    } else {
        gd.bt = std::min(g->bt, g->T); gd.bh = std::min(g->bh, g->H); gd.bw = std::min(g->bw, g->W);
        gd.nH = (int)ceil_div64(g->H, g->bh);
        gd.nW = (int)ceil_div64(g->W, g->bw);
    }
    gd.S = (int)S;
    gd.n_blocks = nb;
    int64_t chunks = n_tensors ? 0 : ceil_div64(S, INDEX_CHUNK);
    for (int i = 0; i < n_tensors; ++i) chunks = std::max(chunks, ceil_div64(S * Hh * (D * (cd.in_bf16[i] ? 2 : 4) / 16), chunk_pieces(inverse)));
    auto kfn = inverse ? permute_rows_kernel<true, false> : build_index ? permute_rows_kernel<false, true> : permute_rows_kernel<false, false>;
    VMOBA_PROFILE_BEGIN(3, st);
    constexpr int64_t PER_LAUNCH = 1 << 23;             // (a launch holds less than 2^32 threads)
    for (int64_t c0 = 0; c0 < chunks; c0 += PER_LAUNCH) {
        const dim3 grid((unsigned)std::min(PER_LAUNCH, chunks - c0), (unsigned)(n_tensors ? B : 1), (unsigned)std::max(n_tensors, 1));
        kfn<<<grid, dim3(256), 0, st>>>(gd, cd, perm, inv_perm, blk_off, Hh, D, (unsigned)c0);
    }
    VMOBA_PROFILE_END(3, st);
    VMOBA_CHECK_LAUNCH();
    return VMOBA_OK;
}

extern "C" const char* vmoba_status_string(int status) {
    switch (status) {
        case VMOBA_OK: return "ok";
        case VMOBA_ERR_INVALID_ARG: return "invalid argument";
        case VMOBA_ERR_UNSUPPORTED: return "unsupported configuration";
        case VMOBA_ERR_WORKSPACE: return "workspace too small";
        case VMOBA_ERR_CAPACITY: return "nnz capacity exceeded";
        case VMOBA_ERR_HIP: return "HIP error";
        default: return "unknown status";
    }
}
