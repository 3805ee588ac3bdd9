"""Sizes at which the tile kernels and the selection kernels can go wrong: edges of tiles, remainders, the smallest of a
range.  Most cases run a whole layer against the CPU oracle (bounds: tests/gpu_util.py)."""
import math

import numpy as np
import pytest
import torch

from oracle import vmoba_oracle as vo
from paper_2506_23858_amd import binding as vb, synth
from tests import gpu_util as gu
from tests.test_gpu_parity import compare_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [2, 32, 33, 64, 65, 97, 199])
def test_f32_matrix_kernels_at_tile_edges(chunk, D):
    """Blocks of one key (199 + 1), of two, of one 32-key chunk, one key more, one and two 64-key runs, and lists that end inside and at the
    end of a 64-query chunk and of a 128-query tile (200 queries, thresholds that keep a part or all of them)."""
    grid, S = (1, 8, 25), 200
    Q, K, V, dO = (synth.iid_normal(900 + i, (1, S, 2, D)) for i in range(4))
    for tau, kv_in_place in ((0.6, False), (1.0, True)):
        g, _ = compare_layer(Q, K, V, dO, grid, (0, 0, 0), chunk, tau, torch.float32, f"f32-edges-{chunk}", kv_in_place=kv_in_place)
        assert not gu.multiplies_split_operands(g["plan"])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [2, 31, 33, 64, 97, 129, 161, 200])
def test_bf16_backward_kernels_at_tile_edges(chunk, D):
    """Blocks that end one key before and after a 32-key group, a 64-key chunk, a 128-key run and its tail of at most 32 keys (also a run
    whose second half has no keys); lists of a few entries and of 400 (longer than the ring of eight half-chunks, ending
    inside one), keys rearranged and in place."""
    grid, S = (1, 8, 50), 400
    Q, K, V, dO = (synth.to_bf16_grid(synth.blurred_noise(940 + i, grid, 2, D, 1.0)) for i in range(4))
    for tau, kv_in_place in ((0.3, True), (1.0, False)):
        compare_layer(Q, K, V, dO, grid, (0, 0, 0), chunk, tau, torch.bfloat16, f"bf16-edges-{chunk}", kv_in_place=kv_in_place)


@pytest.mark.parametrize("chunk,topk", [(1, 2), (1, 3), (2, 1), (2, 256)])
def test_bf16_backward_of_many_blocks_and_few_pairs(chunk, topk):
    """512 and 256 blocks: the slots of the dK/dV kernel need more room than the tile list leaves, and
    less.  (Every query keeps two keys at least: of a single one dQ is 0 and dK nothing but rounding.)"""
    grid, S = (1, 16, 32), 512
    Q, K, V, dO = (synth.to_bf16_grid(synth.iid_normal(1140 + i, (1, S, 3, 64))) for i in range(4))
    compare_layer(Q, K, V, dO, grid, (0, 0, 0), chunk, 0.4, torch.bfloat16, f"slots-{chunk}", mode=1, topk=topk)


@pytest.mark.parametrize("mode,topk", [(1, 1), (1, 5), (1, 1000), (2, 0), (0x101, 3)])
@pytest.mark.parametrize("chunk", [48, 43, 42, 6, 5, 3, 2, 1])
def test_local_selections_at_column_counts(chunk, mode, topk):
    """Per-query selections with 8, 9, 10, 64, 77, 128, 192 and 384 blocks: columns that fill a lane's share, exceed it by one and by a few, rows
    held by one to eight lanes, 16-byte aligned or not; keep one, several, all blocks, and the query's own block as well."""
    grid, S = (1, 16, 24), 384
    Q, K, V = (synth.to_bf16_grid(synth.iid_normal(970 + i, (1, S, 2, 64))) for i in range(3))
    compare_layer(Q, K, V, None, grid, (0, 0, 0), chunk, 0.4, torch.bfloat16, f"local-{chunk}", mode=mode, topk=topk)


@pytest.mark.parametrize("blocks", [63, 64, 65, 128, 257, 512])
def test_pair_lists_longer_than_a_window(blocks):
    """Every pair kept: 64 queries hold one entry window less a row, exactly one, one and a row, two, four and a row, eight; the mass cut of more than
    256 blocks counts its histogram by another kernel and has to agree that the whole pool is kept."""
    S = 512
    chunk = -(-S // blocks)
    grid = (1, 1, blocks * chunk)
    Q, K, V = (synth.to_bf16_grid(synth.iid_normal(1020 + i, (1, blocks * chunk, 1, 64))) for i in range(3))
    for tau, mode, topk in ((1.0, 0, 0), (0.4, 1, blocks)):
        compare_layer(Q, K, V, None, grid, (0, 0, 0), chunk, tau, torch.bfloat16, f"lists-{blocks}", mode=mode, topk=topk)


def check_heads(case, g, Q, K, V, dO, heads, scale=None, dtype=torch.float32, b=0):
    """Attention outputs of some heads of a batch element against the oracle under the GPU's own mask."""
    perm = g["perm"]
    scale = 1.0 / math.sqrt(Q.shape[3]) if scale is None else scale
    for h in heads:
        q, k, v, d = (x[b, perm, h].astype(np.float64) for x in (Q, K, V, dO))
        m = g["mask"][b, h]
        O, LSE = vo.masked_attention_fwd(q, k, v, m, g["blk_off"], scale)
        dQ, dK, dV = vo.masked_attention_bwd(q, k, v, m, g["blk_off"], scale, d)
        live = np.isfinite(LSE)
        gu.check_output(case, "LSE", g["LSE"][b, h][live], LSE[live], dtype)
        for name, ref in (("Op", O), ("dQp", dQ), ("dKp", dK), ("dVp", dV)):
            gu.check_output(case, name.rstrip("p"), g[name][b, h], ref, dtype)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [31, 33, 97, 129, 300])
def test_f32_split_kernels_at_tile_edges(chunk, D):
    """float32 calls large enough for the kernels on split operands: blocks that end around a 32-key group and around a run of 128 keys
    (one key, and one wavefront's keys and one more, in the last run), lists that end inside a 32-query chunk."""
    grid, S, heads = (1, 48, 50), 2400, 24 if D == 64 else 8
    Q, K, V, dO = (synth.iid_normal(1000 + i, (1, S, heads, D)) for i in range(4))
    g = gu.run_gpu(Q, K, V, dO, grid, (0, 0, 0), chunk, 0.95 if chunk < 200 else 0.4, torch.float32, kv_in_place=chunk == 97)
    assert gu.multiplies_split_operands(g["plan"])
    check_heads(f"f32-split-{chunk}-{D}", g, Q, K, V, dO, (0, heads - 1))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("scale", [-0.07, 0.0])
def test_f32_split_kernels_take_a_scale_of_any_sign(scale, D):
    """Scores that count downwards and scores that do not count, with keys past the block's end in the last 32-key group (blocks of 97 and 300)."""
    grid, S, heads = (1, 48, 50), 2400, 24 if D == 64 else 8
    Q, K, V, dO = (synth.iid_normal(1030 + i, (1, S, heads, D)) for i in range(4))
    for chunk, tau in ((97, 0.95), (300, 0.4)):
        g = gu.run_gpu(Q, K, V, dO, grid, (0, 0, 0), chunk, tau, torch.float32, softmax_scale=scale)
        assert gu.multiplies_split_operands(g["plan"])
        check_heads(f"f32-split-scale-{scale}-{chunk}-{D}", g, Q, K, V, dO, (0, heads - 1), scale)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("scale", [-0.09, 0.0])
def test_bf16_kernels_take_a_scale_of_any_sign(scale, D):
    """The same for the bfloat16 kernels: blocks of one 32-key group and less, of one and a part, of whole groups, of a 64-key chunk and a part."""
    grid, S, heads = (1, 8, 50), 400, 2
    Q, K, V, dO = (synth.to_bf16_grid(synth.iid_normal(1040 + i, (1, S, heads, D))) for i in range(4))
    for chunk, kv_in_place in ((20, False), (33, True), (64, False), (97, True)):
        g = gu.run_gpu(Q, K, V, dO, grid, (0, 0, 0), chunk, 0.6, torch.bfloat16, softmax_scale=scale, kv_in_place=kv_in_place)
        check_heads(f"bf16-scale-{scale}-{chunk}-{D}", g, Q, K, V, dO, range(heads), scale, torch.bfloat16)


def forward_tiles_per_workgroup(g, D):
    """Tiles of a bfloat16 forward call over the workgroups of its persistent kernel (128 channels: 256 queries, one workgroup per compute unit)."""
    TM, per_cu = (256, 1) if D == 128 else (128, 2)
    return int((-(-np.diff(g["blk_ptr"]) // TM)).sum()) / (per_cu * torch.cuda.get_device_properties(0).multi_processor_count)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [20, 96, 97, 160, 161, 224, 300])
def test_bf16_forward_over_many_tiles(chunk, D):
    """Every workgroup of the forward tile kernel walks several tiles (64 heads x 1600 queries): blocks of one to ten key groups --
    as many as a tile counts at least, fewer, an odd and an even number, the last one whole or not -- beside a shorter one at the end, lists that end inside
    a tile, scores so far apart that the running maximum rises often; keys rearranged and in place."""
    grid, S, heads = (1, 32, 50), 1600, 64
    Q, K, V = (synth.to_bf16_grid(synth.iid_normal(1060 + i, (1, S, heads, D))) for i in range(3))
    for scale, tau, kv_in_place in ((None, 0.7, True), (0.5, 1.0, False), (0.5, 1.0, True)):
        g = gu.run_gpu(Q, K, V, None, grid, (0, 0, 0), chunk, tau, torch.bfloat16, softmax_scale=scale, kv_in_place=kv_in_place)
        assert forward_tiles_per_workgroup(g, D) >= 3
        for h in (0, 31, 63) if chunk != 20 else (31,):
            q, k, v = (x[0, g["perm"], h].astype(np.float64) for x in (Q, K, V))
            O, LSE = vo.masked_attention_fwd(q, k, v, g["mask"][0, h], g["blk_off"], 1.0 / math.sqrt(D) if scale is None else scale)
            live = np.isfinite(LSE)
            gu.check_output(f"bf16-tiles-{chunk}-{D}", "LSE", g["LSE"][0, h][live], LSE[live], torch.bfloat16)
            gu.check_output(f"bf16-tiles-{chunk}-{D}", "O", g["Op"][0, h], O, torch.bfloat16)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [390, 480, 512])
def test_bf16_forward_in_place_over_many_long_tiles(chunk, D):
    """Blocks of 13, 15 and 16 key groups found through kv_rows, each workgroup walking at least three tiles: the row numbers of a tile are requested while
    two earlier ones are worked on.  Every head gives the bits that rearranged keys give; some against the oracle."""
    grid, S, heads, tau = (1, 30, 52), 1560, 48, 0.9
    Q, K, V = (synth.to_bf16_grid(synth.iid_normal(1080 + i, (1, S, heads, D))) for i in range(3))
    g, r = (gu.run_gpu(Q, K, V, None, grid, (0, 0, 0), chunk, tau, torch.bfloat16, kv_in_place=kv, q_in_place=True) for kv in (True, False))
    assert forward_tiles_per_workgroup(g, D) >= 3
    assert np.array_equal(g["mask"], r["mask"]) and np.array_equal(g["LSE"], r["LSE"]) and np.array_equal(g["O"], r["O"])
    for h in (0, 24, 47):
        q, k, v = (x[0, g["perm"], h].astype(np.float64) for x in (Q, K, V))
        O, LSE = vo.masked_attention_fwd(q, k, v, g["mask"][0, h], g["blk_off"], 1.0 / math.sqrt(D))
        live = np.isfinite(LSE)
        gu.check_output(f"bf16-in-place-{chunk}-{D}", "LSE", g["LSE"][0, h][live], LSE[live], torch.bfloat16)
        gu.check_output(f"bf16-in-place-{chunk}-{D}", "O", g["Op"][0, h], O, torch.bfloat16)


@pytest.mark.parametrize("kv_in_place", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("chunk", [32, 64, 96, 128, 160])
def test_bf16_forward_keeps_an_infinity_of_a_block_of_whole_groups(chunk, D, kv_in_place):
    """An infinite channel in the last value row of a block of 1 to 5 key groups, without a key missing in the last one: infinite for the queries
    that keep the block (NaN if it is the last one they keep: the merge meets it again with weight 0), and nothing else changes."""
    grid, S, heads, channel = (1, 1, 3 * chunk), 3 * chunk, 4, 5
    Q, K, V = (synth.to_bf16_grid(synth.iid_normal(1090 + i, (1, S, heads, D))) for i in range(3))
    finite = gu.run_gpu(Q, K, V, None, grid, (0, 0, 0), chunk, 0.5, torch.bfloat16, kv_in_place=kv_in_place)
    V[0, chunk - 1, :, channel] = np.inf
    g = gu.run_gpu(Q, K, V, None, grid, (0, 0, 0), chunk, 0.5, torch.bfloat16, kv_in_place=kv_in_place)
    keeps, others = g["mask"][0, :, :, 0], g["mask"][0, :, :, 1:].any(-1)
    assert np.array_equal(g["mask"], finite["mask"]) and np.array_equal(g["LSE"], finite["LSE"])
    assert (keeps & others).any() and not keeps.all() and np.all(g["Op"][0, ..., channel][keeps & others] == np.inf)
    assert not np.isfinite(g["Op"][0, ..., channel][keeps]).any()
    g["Op"][0, ..., channel][keeps] = finite["Op"][0, ..., channel][keeps]
    assert np.array_equal(g["Op"], finite["Op"])


@pytest.mark.parametrize("kv_in_place", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("grid,block,chunk", [
    ((1, 8, 50), (0, 0, 0), 1), ((1, 8, 50), (0, 0, 0), 31), ((1, 8, 50), (0, 0, 0), 32), ((1, 8, 50), (0, 0, 0), 33),
    ((1, 8, 50), (0, 0, 0), 63), ((1, 8, 50), (0, 0, 0), 64),
    ((5, 9, 9), (4, 8, 8), 0),         # 50 keys on average: one block of 256, others of 64, 32, 8, 4 and 1
])
def test_bf16_forward_of_short_blocks(grid, block, chunk, D, kv_in_place):
    """Calls whose usual block has at most 64 keys skip what groups without a key have to do: blocks of one key, around one and two whole groups, and
    short ones beside one of eight groups, over many tiles of 64 heads."""
    S, heads = grid[0] * grid[1] * grid[2], 64
    Q, K, V = (synth.to_bf16_grid(synth.iid_normal(1100 + i, (1, S, heads, D))) for i in range(3))
    for scale, tau in ((None, 0.6), (0.5, 0.95)):
        g = gu.run_gpu(Q, K, V, None, grid, block, chunk, tau, torch.bfloat16, softmax_scale=scale, kv_in_place=kv_in_place)
        for h in (0, 31, 63):
            q, k, v = (x[0, g["perm"], h].astype(np.float64) for x in (Q, K, V))
            O, LSE = vo.masked_attention_fwd(q, k, v, g["mask"][0, h], g["blk_off"], 1.0 / math.sqrt(D) if scale is None else scale)
            live = np.isfinite(LSE)
            gu.check_output(f"bf16-short-{chunk}-{D}", "LSE", g["LSE"][0, h][live], LSE[live], torch.bfloat16)
            gu.check_output(f"bf16-short-{chunk}-{D}", "O", g["Op"][0, h], O, torch.bfloat16)


def test_bf16_forward_takes_query_rows_far_apart():
    """Rows of Q 16 MB and more apart (their offsets do not fit 32 bits) give the same bits as rows that are neighbours."""
    grid, S, D, pitch = (1, 8, 40), 320, 128, (1 << 23) + 8
    Q, K, V = (gu.to_dev(synth.to_bf16_grid(synth.iid_normal(1070 + i, (1, S, 1, D))), torch.bfloat16) for i in range(3))
    wide = torch.empty((S - 1) * pitch + D, dtype=torch.bfloat16, device="cuda").as_strided((1, S, 1, D), (S * pitch, pitch, D, 1))
    wide.copy_(Q)
    plan = vb.LayerPlan(1, 1, D, grid, chunk=64, tau=0.7, dtype=torch.bfloat16, need_bwd=False, q_in_place=True)
    O = [plan.forward(q, K, V).clone() for q in (Q, wide)]
    torch.cuda.synchronize()
    assert torch.equal(*O) and float(O[0].float().abs().max()) > 0


def test_f32_split_kernels_hand_infinities_to_the_float32_ones():
    """An infinity has no terms to split into: an infinite channel of one value row makes that channel of every query that keeps the key
    infinite (NaN where the merge meets it again with weight 0), and nothing else, as it does in a call of any size."""
    grid, S, heads, D = (1, 48, 50), 2400, 8, 128
    Q, K, V, dO = (synth.iid_normal(1010 + i, (1, S, heads, D)) for i in range(4))
    ref = gu.run_gpu(Q, K, V, None, grid, (0, 0, 0), 300, 0.4, torch.float32)
    assert gu.multiplies_split_operands(ref["plan"])
    V[0, 777, 3, 5] = np.inf
    g = gu.run_gpu(Q, K, V, None, grid, (0, 0, 0), 300, 0.4, torch.float32)
    keeps = g["mask"][0, 3][:, 777 // 300]
    assert keeps.any() and not keeps.all()
    assert (g["Op"][0, 3][keeps, 5] == np.inf).any() and not np.isfinite(g["Op"][0, 3][keeps, 5]).any()
    g["Op"][0, 3][keeps, 5] = ref["Op"][0, 3][keeps, 5]
    gu.check_output("f32-split-inf", "O", g["Op"], ref["Op"], torch.float32)


def relative_error(got, ref):
    return float(np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("powers", [(60, 55), (110, 0), (0, 110), (118, 0)])
def test_f32_split_kernels_on_small_magnitudes(powers):
    """dO and V scaled by powers of two: everything they enter scales along, exactly but for what falls below the smallest normal number (last
    bit 2^-149: 1e-7 of values of 2^-126 and up).  Operands below 2^-100 have no three terms of eight bits: such a call takes the
    float32 kernels, whose sums differ from the others' by up to 1e-6."""
    grid, S, heads, D = (1, 48, 50), 2400, 8, 128
    Q, K, V, dO = (synth.iid_normal(1050 + i, (1, S, heads, D)) for i in range(4))
    do_pow, v_pow = powers
    a, b = (gu.run_gpu(Q, K, v, d, grid, (0, 0, 0), 300, 0.4, torch.float32)
            for v, d in ((V, dO), (V * np.float32(2.0 ** -v_pow), dO * np.float32(2.0 ** -do_pow))))
    assert gu.multiplies_split_operands(a["plan"])
    for name, power in (("Op", v_pow), ("dVp", do_pow), ("dQp", do_pow + v_pow), ("dKp", do_pow + v_pow)):
        err = relative_error(b[name].astype(np.float64) * 2.0 ** power, a[name].astype(np.float64))
        print(f"   {name}: {err:.2e}", flush=True)
        assert err <= (1e-7 if max(powers) < 100 else 1e-6), (name, err)


def test_f32_split_kernels_on_small_weights():
    """A key with weights of about 2^-124 in every row that keeps it: its dV and dK are sums of such numbers alone and keep float32's relative
    precision (1e-4: the exponent itself is exact to 2^-17 there, 5e-6 of the weight; eight bits of a weight are 4e-3)."""
    grid, S, heads, D = (1, 48, 50), 2400, 8, 128
    Q, K, V, dO = (synth.iid_normal(1060 + i, (1, S, heads, D)) for i in range(4))
    Q[..., 0], K[..., 0] = 16.0, 0.0
    K[:, 777] = 0.0
    K[:, 777, :, 0] = -55.0
    g = gu.run_gpu(Q, K, V, dO, grid, (0, 0, 0), 300, 1.0, torch.float32)
    assert gu.multiplies_split_operands(g["plan"])
    pos, scale = int(g["inv_perm"][777]), 1.0 / math.sqrt(D)
    for h in (0, heads - 1):
        q, k, v, d = (x[0, g["perm"], h].astype(np.float64) for x in (Q, K, V, dO))
        O, LSE = vo.masked_attention_fwd(q, k, v, g["mask"][0, h], g["blk_off"], scale)
        w = np.exp(scale * q @ k[pos] - LSE)
        assert 2.0 ** -126 < w.min() and w.max() < 2.0 ** -120
        dS = w * (d @ v[pos] - (d * O).sum(1))
        errs = relative_error(g["dVp"][0, h, pos], w @ d), relative_error(g["dKp"][0, h, pos], scale * dS @ q)
        print("   dV %.2e dK %.2e" % errs, flush=True)
        assert max(errs) <= 1e-4


@pytest.mark.parametrize("power", [11, 20])
@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_kernels_on_rows_of_different_magnitudes(power, D):
    """One row of dO far smaller than the others of its head: that query's dQ scales along, the others' rows stay.  (1e-6: what two kinds of kernels
    differ by; the test below has one kind and asks for the bits.)"""
    grid, S, heads = (1, 48, 50), 2400, 24 if D == 64 else 8
    Q, K, V, dO = (synth.iid_normal(1090 + i, (1, S, heads, D)) for i in range(4))
    small = dO.copy()
    small[0, 777] *= np.float32(2.0 ** -power)
    a, b = (gu.run_gpu(Q, K, V, d, grid, (0, 0, 0), 300, 0.4, torch.float32) for d in (dO, small))
    assert gu.multiplies_split_operands(a["plan"])
    pos = int(a["inv_perm"][777])
    kept = a["mask"][0][:, pos].any(-1)
    assert kept.any()
    err = relative_error(b["dQp"][0, kept, pos].astype(np.float64) * 2.0 ** power, a["dQp"][0, kept, pos].astype(np.float64))
    rest = [np.delete(g["dQp"], pos, 2) for g in (b, a)]
    print("   dQ %.2e, other rows %.2e" % (err, relative_error(rest[0], rest[1].astype(np.float64))), flush=True)
    assert err <= 1e-6 and relative_error(rest[0], rest[1].astype(np.float64)) <= 1e-6


@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_kernels_on_rows_far_apart_in_magnitude(D):
    """One row of dO 2^-20 of the others of its head: the call stays on the split kernels -- the other queries' dQ have the bits of the call with ordinary
    rows, which the sums of the kernels on the float32 instruction do not give -- and that query's dQ scales along exactly."""
    grid, S, heads = (1, 48, 50), 2400, 24 if D == 64 else 8
    Q, K, V, dO = (synth.iid_normal(1090 + i, (1, S, heads, D)) for i in range(4))
    small = dO.copy()
    small[0, 777] *= np.float32(2.0 ** -20)
    a, b = (gu.run_gpu(Q, K, V, d, grid, (0, 0, 0), 300, 0.4, torch.float32) for d in (dO, small))
    assert gu.multiplies_split_operands(a["plan"])
    b["dQ"][0, 777] *= np.float32(2.0 ** 20)
    assert a["dQ"][0, 777].any() and np.array_equal(a["dQ"], b["dQ"])


@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_kernels_on_channels_of_different_magnitudes(D):
    """A channel 2^-24 of the others of its rows, of each tensor in turn: what it alone decides -- a channel of O (of V), dV (of dO), dK (of Q), dQ (of K) --
    scales along exactly, as float32 sums do, and nothing else changes.  (In the products that would couple it to the rest, the other operand's channel is 0.)"""
    grid, S, heads = (1, 48, 50), 2400, 24 if D == 64 else 8
    Q, K, V, dO = (synth.iid_normal(1100 + i, (1, S, heads, D)) for i in range(4))
    dO[..., 5] = V[..., 6] = K[..., 7] = Q[..., 8] = 0.0
    small = [x.copy() for x in (Q, K, V, dO)]
    for x, c in zip(small, (7, 8, 5, 6)):
        x[..., c] *= np.float32(2.0 ** -24)
    a, b = (gu.run_gpu(*x, grid, (0, 0, 0), 300, 0.4, torch.float32) for x in ((Q, K, V, dO), small))
    assert gu.multiplies_split_operands(a["plan"]) and np.array_equal(a["mask"], b["mask"])
    for name, c in (("O", 5), ("dV", 6), ("dK", 7), ("dQ", 8)):
        b[name][..., c] *= np.float32(2.0 ** 24)
        err = relative_error(b[name][..., c], a[name][..., c].astype(np.float64))
        print(f"   {name}: {err:.2e}", flush=True)
        assert a[name][..., c].any() and np.array_equal(a[name], b[name]), (name, err)


@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_kernels_on_a_large_value_row(D):
    """One row of V 2^12 times the others: O and dQ of the queries that do not keep its block have the bits they have without it."""
    grid, S, heads = (1, 48, 50), 2400, 24 if D == 64 else 8
    Q, K, V, dO = (synth.iid_normal(1110 + i, (1, S, heads, D)) for i in range(4))
    large = V.copy()
    large[0, 777] *= 4096.0
    a, b = (gu.run_gpu(Q, K, v, dO, grid, (0, 0, 0), 300, 0.4, torch.float32) for v in (V, large))
    assert gu.multiplies_split_operands(a["plan"])
    others = ~a["mask"][0, :, :, 777 // 300]                       # (perm is the identity here)
    assert others.any() and not others.all()
    for name in ("Op", "dQp"):
        err = relative_error(b[name][0][others], a[name][0][others].astype(np.float64))
        print(f"   {name}: {err:.2e}", flush=True)
        assert np.array_equal(a[name][0][others], b[name][0][others]), (name, err)


@pytest.mark.parametrize("heavy", [3, 2397])
@pytest.mark.parametrize("zero", ["dO", "Q"])
def test_f32_split_kernels_on_zero_rows(zero, heavy):
    """A key whose one large weight belongs to a query with a row of zeros in dO (a token that the loss masks), or in Q, and whose other weights are near 2^-36: its
    dV (its dK) consists of those alone and keeps their relative precision, wherever in the list that query comes.  (Exponents of up to 64 are exact to 2^-18 in
    float32: 3e-6 of a weight; 1e-5 with the rounding of the LSE.)"""
    grid, S, heads, D = (1, 48, 50), 2400, 8, 128
    Q, K, V, dO = (synth.iid_normal(1120 + i, (1, S, heads, D)) for i in range(4))
    scale, kx = 1.0 / math.sqrt(D), 777
    Q[..., 0], K[..., 0], Q[..., 1], K[..., 1] = 16.0, 0.0, 0.0, 0.0
    K[:, kx] = 0.0
    K[:, kx, :, 0], K[:, kx, :, 1] = -12.0, 16.0
    if zero == "dO":
        Q[:, heavy, :, 1] = 19.0
        dO[:, heavy] = 0.0
    else:
        Q[:, heavy] = 0.0
    g = gu.run_gpu(Q, K, V, dO, grid, (0, 0, 0), 300, 1.0, torch.float32)
    assert gu.multiplies_split_operands(g["plan"])
    worst = 0.0
    for h in (0, heads - 1):
        q, k, v, d = (x[0, :, h].astype(np.float64) for x in (Q, K, V, dO))
        O, LSE = vo.masked_attention_fwd(q, k, v, g["mask"][0, h], g["blk_off"], scale)
        w = np.exp(scale * q @ k[kx] - LSE)
        rest = np.delete(w, heavy)
        assert rest.max() < 2.0 ** -32 and w[heavy] > 2.0 ** -12
        dS = w * (d @ v[kx] - (d * O).sum(1))
        errs = relative_error(g["dVp"][0, h, kx], w @ d), relative_error(g["dKp"][0, h, kx], scale * dS @ q)
        print("   dV %.2e dK %.2e" % errs, flush=True)
        worst = max(worst, errs[0] if zero == "dO" else 0.0, errs[1])
    assert worst <= 1e-5


@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_kernels_read_keys_through_their_row_numbers_only(D):
    """kv_rows may name any row of K and V: their last S rows of 2 S here, behind rows 2^-12 and 2^12 of them.  Same bits as with those rows alone."""
    grid, S, heads, chunk, tau = (1, 48, 50), 2400, 24 if D == 64 else 8, 300, 0.4
    Q, K, V, dO = (gu.to_dev(synth.iid_normal(1130 + i, (1, S, heads, D)), torch.float32) for i in range(4))
    plan = vb.LayerPlan(1, heads, D, grid, (0, 0, 0), chunk, tau, torch.float32, kv_in_place=True)
    assert gu.multiplies_split_operands(plan)
    plan.forward(Q, K, V)
    plan.backward(dO)
    torch.cuda.synchronize()
    want = {n: getattr(plan, n).clone() for n in ("O", "LSE", "dQ", "dK", "dV", "mask")}
    rows = plan.perm + S
    for power in (-12, 12):
        wide = [torch.cat([x * 2.0 ** power, x], 1) for x in (K, V)]
        for n in want:
            getattr(plan, n).zero_()
        vb.vmoba_select(1, heads, S, D, plan.nb, plan.blk_off, Q, wide[0], tau, plan.score_scale, plan.mode, 0, plan.Bmean, plan.P, plan.mask, plan.blk_ptr,
                        plan.q_idx, plan.row_ptr, plan.col_idx, plan.pair_pos, plan.cap, plan.k_out, plan.theta, plan.dev_status, plan.ws_select,
                        query_pos=plan.inv_perm, kv_rows=rows)
        lists = (plan.blk_ptr, plan.q_idx, plan.row_ptr, plan.pair_pos, plan.cap, plan.softmax_scale)
        vb.vmoba_attn_fwd(1, heads, S, D, plan.nb, plan.blk_off, Q, *wide, *lists, plan.O, plan.LSE, plan.ws_attn, kv_rows=rows)
        vb.vmoba_attn_bwd(1, heads, S, D, plan.nb, plan.blk_off, Q, *wide, plan.O, plan.LSE, dO, *lists, plan.dQ, plan.dK, plan.dV, plan.ws_attn,
                          key_rows=plan.perm, kv_rows=rows)
        torch.cuda.synchronize()
        for n, x in want.items():
            assert torch.equal(getattr(plan, n), x), (power, n)


@pytest.mark.parametrize("layout", [{}, {"fused_io": True}, {"q_in_place": True}, {"kv_in_place": True}])
@pytest.mark.parametrize("D", [64, 128])
def test_f32_split_kernels_in_every_layout(D, layout):
    """Two videos, Q, K and V views of one packed projection: operands split from block order and from the caller's rows, dO with and
    without its block-order copy, dK and dV written through a row map."""
    grid, block, heads = (4, 15, 20), (2, 7, 9), 12 if D == 64 else 6
    S = grid[0] * grid[1] * grid[2]
    Q, K, V, dO = (synth.blurred_noise(1070 + i, (2 * grid[0],) + grid[1:], heads, D, 1.0).reshape(2, S, heads, D) for i in range(4))
    g = gu.run_gpu(Q, K, V, dO, grid, block, 0, 0.9, torch.float32, packed=True, **layout)
    assert gu.multiplies_split_operands(g["plan"])
    for b, h in ((0, 0), (1, heads - 1)):
        check_heads(f"f32-split-layout-{'-'.join(layout)}-{D}", g, Q, K, V, dO, (h,), b=b)


@pytest.mark.parametrize("chunk,layout", [(97, {}), (129, {"kv_in_place": True}), (300, {"fused_io": True})])
def test_f32_calls_of_values_that_do_not_split_and_the_next_one(chunk, layout):
    """One infinite value of dO in one head, one NaN of V in another: the whole call is handed to the float32 kernels, backward included, which
    then walk a run table of 128 keys in halves of 64.  What the two values do not enter matches the oracle;
    the call after it, of finite values in the same buffers, has the bits of the call before."""
    grid, S, heads, D = (1, 48, 50), 2400, 8, 128
    Q, K, V, dO = (synth.iid_normal(1080 + i, (1, S, heads, D)) for i in range(4))
    plan = vb.LayerPlan(1, heads, D, grid, (0, 0, 0), chunk, 0.95 if chunk < 200 else 0.4, torch.float32, **layout)
    assert gu.multiplies_split_operands(plan)

    def run(V, dO):
        plan.forward(*(gu.to_dev(x, torch.float32) for x in (Q, K, V)))
        plan.backward(gu.to_dev(dO, torch.float32))
        torch.cuda.synchronize()
        assert int(plan.dev_status.item()) == 0
        return {n: gu.np32(getattr(plan, n))[0] for n in ("O", "dQ", "dK", "dV")}

    before = run(V, dO)
    assert all(np.isfinite(x).all() for x in before.values())
    q_bad, k_bad, dO_bad, V_bad = 1234, 777, dO.copy(), V.copy()
    dO_bad[0, q_bad, 2, 9] = np.inf
    V_bad[0, k_bad, 5, 7] = np.nan
    got = run(V_bad, dO_bad)
    mask = gu.unpack_mask(plan.mask.cpu().numpy(), plan.nb)[0]             # perm is the identity here: query and key ids are tokens
    touched = {n: np.zeros((S, heads, D), bool) for n in before}
    block = np.arange(S) // chunk
    keys = mask[2, q_bad][block]                                           # keys that the query of the infinite dO meets
    queries = mask[5][:, k_bad // chunk]                                   # queries that meet the key of the NaN
    touched["dQ"][q_bad, 2] = touched["dK"][keys, 2] = True
    touched["dV"][keys, 2, 9] = True
    touched["O"][queries, 5, 7] = touched["dQ"][queries, 5] = True
    touched["dK"][mask[5][queries].any(0)[block], 5] = True
    for n, x in before.items():
        t = touched[n]
        if n in ("dQ", "dK"):                                              # (a zero weight may spare single channels of O and dV)
            assert t.any() and not np.isfinite(got[n][t]).any(), n
        gu.check_output(f"f32-split-not-finite-{chunk}", n, got[n][~t], x[~t], torch.float32)
    after = run(V, dO)
    for n in before:
        assert np.array_equal(before[n], after[n]), n


@pytest.mark.parametrize("S,chunk,mode,topk", [
    (256, 2, 0, 0), (256, 2, 0x103, 9), (257, 2, 0, 0),       # 128 blocks: the most the one-launch cut takes, and one more
    (4096, 512, 0, 0), (4096, 512, 4, 0), (4097, 512, 0, 0),  # 4096 rows of 8 values, and one row more
    (331, 5, 0x100, 0), (331, 5, 3, 20), (331, 5, 4, 0),      # pools of 331 x 67 values: only the first head's is 16-byte aligned
    (3, 3, 0, 0), (67, 1, 3, 3),                              # one block; as many blocks as queries
])
def test_cut_among_equal_values(S, chunk, mode, topk):
    """Query rows and key blocks that repeat, so that runs of equal values cross the cut: it keeps the k best of the GPU's own P, equal ones by
    query, then block, and k is the shortest prefix that reaches tau of the mass (or topk * S)."""
    heads, D, tau = 3, 64, 0.37
    nb = -(-S // chunk)
    Q, K, V = (synth.iid_normal(1090 + i, (1, S, heads, D)) for i in range(3))
    Q = np.ascontiguousarray(Q[:, np.arange(S) // 7 * 7 % S])
    K = np.ascontiguousarray(K[:, np.arange(S) % (max(1, nb // 3) * chunk)])
    g = gu.run_gpu(Q, K, V, None, (1, 1, S), (0, 0, 0), chunk, tau, torch.float32, mode=mode, topk=topk)
    total = 1.0 if mode == 4 else float(S)
    cut_ties = 0
    for h in range(heads):
        p = g["P"][0, h].reshape(-1)
        order = np.lexsort((np.arange(p.size), -p))
        mass = np.cumsum(p[order], dtype=np.float64)
        if mode & 0xff == 3:
            k = topk * S
        else:
            k = int(np.searchsorted(mass, np.float32(tau) * total)) + 1
            # (both sides' sums are exact to far less than 1e-6: no prefix may end that close)
            assert np.abs(mass[max(0, k - 2):k] - np.float32(tau) * total).min() > 1e-6 * total
        keep = np.zeros(p.size, bool)
        keep[order[:k]] = True
        cut_ties += bool(k < p.size and p[order[k]] == p[order[k - 1]])
        keep = keep.reshape(S, nb)
        if mode & 0x100:
            keep[np.arange(S), np.arange(S) // chunk] = True
        else:
            assert int(g["k"][0, h]) == k
        assert np.array_equal(g["mask"][0, h], keep), (h, k, int((g["mask"][0, h] != keep).sum()))
        gu.check_lists(g, 0, h)
    assert cut_ties or nb == 1 or S <= 67


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tile_list_of_many_heads(dtype):
    """600 heads x 16 blocks, past the number from which on the heads' tiles are counted in a launch of their own: the first, a middle and the
    last head."""
    S, heads, D = 64, 600, 64
    Q, K, V, dO = (synth.to_bf16_grid(synth.iid_normal(1100 + i, (1, S, heads, D))) for i in range(4))
    g = gu.run_gpu(Q, K, V, dO, (1, 1, S), (0, 0, 0), 4, 0.5, dtype)
    check_heads(f"many-heads-{gu.dtype_name(dtype)}", g, Q, K, V, dO, (0, 299, heads - 1), dtype=dtype)


@pytest.mark.parametrize("Hh,D,S,tin,tout", [
    (1, 64, 1, torch.bfloat16, torch.bfloat16), (1, 64, 331, torch.bfloat16, torch.bfloat16),     # 33 positions of 8 pieces in a workgroup's 256
    (3, 64, 97, torch.float32, torch.float32), (5, 128, 67, torch.float32, torch.bfloat16),       # positions that straddle workgroups
    (16, 128, 8, torch.bfloat16, torch.bfloat16), (17, 128, 31, torch.bfloat16, torch.bfloat16),  # one position per workgroup, and a piece row more
    (40, 128, 13, torch.float32, torch.float32),                                                  # a position in five workgroups
])
def test_partition_across_workgroup_borders(Hh, D, S, tin, tout):
    """Moves and index arrays where workgroups' runs of pieces and the rows of a position do not line up; two batch elements, two tensors of
    their own type, a forward move that reads perm, its inverse, and a call for the index arrays alone."""
    g = vb.make_grid(1, 1, S, 0, 0, 0, max(1, S // 3)) if S < 300 else vb.make_grid(1, 3, S, 1, 2, 7)
    S, nb = vb.vmoba_partition_dims(g)
    perm, inv_perm, blk_off = vo.partition_index(g.T, g.H, g.W, g.bt, g.bh, g.bw, g.chunk)
    x, y = torch.randn(2, S, Hh, D, device="cuda").to(tin), torch.randn(2, S, Hh, D, device="cuda").to(torch.bfloat16)
    order = torch.from_numpy(perm.astype(np.int64)).cuda()
    i32 = dict(dtype=torch.int32, device="cuda")
    for ins, outs in (([], []), ([x, y], [torch.empty_like(x, dtype=tout), torch.empty_like(y)])):
        idx = [torch.full((n,), -1, **i32) for n in (S, S, nb + 1)]
        vb.vmoba_partition(g, 0, 2, Hh, D, ins, outs, *idx)
        for got, ref in zip(idx, (perm, inv_perm, blk_off)):
            assert np.array_equal(got.cpu().numpy(), ref)
        for a, b in zip(ins, outs):
            assert torch.equal(b, a[:, order].to(b.dtype))
    again = torch.empty_like(outs[0])
    vb.vmoba_partition(g, 0, 2, Hh, D, [x], [again], idx[0], None, None)
    assert torch.equal(again, outs[0])
    back = [torch.empty_like(t) for t in outs]
    vb.vmoba_partition(g, 1, 2, Hh, D, outs, back, idx[0], None, None)
    assert torch.equal(back[0], x.to(tout)) and torch.equal(back[1], y)


@pytest.mark.parametrize("S,chunk,rows", [
    (1024, 16, 8), (1024, 16, 9),     # 512 equal values, the most whose last kept one is looked up, and 576, which are ranked row by row
    (1024, 16, 20),                   # more candidates than the list of a head holds
    (1001, 15, 7), (1001, 15, 1),     # pools of 1001 x 67 values: only the first head's is 16-byte aligned
])
def test_cut_inside_a_run_of_equal_values(S, chunk, rows):
    """Some query rows are zero, so all their values are 1 / N_b, and tau puts the cut in the middle of them: the mask holds the k best of the
    GPU's own P, equal ones by query, then block, with a part of the run kept in every head."""
    heads, D = 3, 64
    Q, K, V = (synth.iid_normal(1120 + i, (1, S, heads, D)) for i in range(3))
    Q[:, 5:5 + rows * (S // rows) - 5:S // rows] = 0.0
    P = gu.run_gpu(Q, K, V, None, (1, 1, S), (0, 0, 0), chunk, 0.5, torch.float32)["P"]
    nb = P.shape[-1]
    equal = P[0, 0, 5, 0]
    for h in range(heads):
        assert int((P[0, h] == equal).sum()) == rows * nb
        tau = (float(P[0, h][P[0, h] > equal].sum(dtype=np.float64)) + 0.5 * rows) / S
        g = gu.run_gpu(Q, K, V, None, (1, 1, S), (0, 0, 0), chunk, tau, torch.float32)
        for i in range(heads):
            p, k = g["P"][0, i].reshape(-1), int(g["k"][0, i])
            order = np.lexsort((np.arange(p.size), -p))
            keep = np.zeros(p.size, bool)
            keep[order[:k]] = True
            assert np.array_equal(g["mask"][0, i].reshape(-1), keep), (h, i, k)
            gu.check_lists(g, 0, i)
        above, kept = int((P[0, h] > equal).sum()), int(g["k"][0, h])
        assert above < kept < above + rows * nb and abs(kept - above - 0.5 * rows * nb) <= 1
