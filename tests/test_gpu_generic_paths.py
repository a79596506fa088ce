"""GPU tests of the kernels outside the 128-wide, 16-position-page bf16 layer: the fp32 projections
(tiles of 16, 32 and 64 rows, K slices of unequal length, widths that fill no tile) and the
matrix-core attention for other head dims, page sizes and fp32 storage, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import GpuRun, check_against_oracle, gemm_path, planes_in_workgroup, say
from paper_2605_21603_amd import binding as B
from workloads import gen

pytestmark = pytest.mark.gpu


def workload(name, dtype, hidden, n_q, n_kv, hd, inter, seqs, page=16, experts=0, top_k=0, seed=40):
    sh = gen.LayerShape(dtype, hidden, n_q, n_kv, hd, inter, n_experts=experts, top_k=top_k, page_size=page)
    cut = seqs[0][0]
    T = sum(q for q, _ in seqs)
    return gen.Workload(name, sh, tuple(seqs), seed, (0, cut, T) if len(seqs) > 1 else (0, T))


def both_schedules(w, data):
    run = GpuRun(w, data)
    y, k, v = run.run(B.sequential())
    if len(w.nano_rows) > 2:
        y1, _, _ = run.run(B.nano_schedule(w.nano_rows, chain=B.MOE_CHAIN if w.shape.n_experts else B.DENSE_CHAIN))
        assert torch.equal(y.view(torch.uint8), y1.view(torch.uint8)), "the split schedule changed bits"
    return y, k, v


# rows at the edges of the 16-, 32- and 64-row tiles; hidden, inter and head widths that leave ragged K slices and column tiles
@pytest.mark.parametrize("rows,hidden,n_q,n_kv,hd,inter", [
    (1, 256, 4, 4, 64, 1024), (16, 68, 2, 1, 32, 100), (17, 132, 3, 1, 8, 52), (33, 36, 1, 1, 64, 260), (64, 256, 4, 2, 64, 4096),
    (65, 260, 4, 2, 64, 8200), (130, 1024, 8, 8, 64, 5124)])
def test_fp32_projections_at_tile_edges(rows, hidden, n_q, n_kv, hd, inter):
    seqs = [(1, 1 + (7 * i) % 40) for i in range(rows)]
    w = workload("f32_%d" % rows, "f32", hidden, n_q, n_kv, hd, inter, seqs)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    # 1e-4 is the layer's fp32 bound; eight shorter chains per output stay well inside one long chain's error
    err = check_against_oracle(w, data, y, k, v)
    say("rows %d: %.2e" % (rows, err))
    assert err < 2e-6


def test_fp32_experts_with_empty_and_long_lists():
    w = workload("f32_moe", "f32", 132, 2, 1, 32, 68, [(1, 3 + i % 9) for i in range(70)], experts=5, top_k=2)
    data = gen.generate(w)
    data["weights"][0]["w_router"][3] = -4.0 * data["weights"][0]["w_router"][0]
    y, k, v = both_schedules(w, data)
    check_against_oracle(w, data, y, k, v)


MIX = [(23, 23), (1, 70), (1, 256), (1, 257), (40, 300), (2, 513), (1, 1)]     # chunk edges, groups that straddle aligned blocks


@pytest.mark.parametrize("dtype,n_q,n_kv,hd,page", [
    ("f32", 4, 4, 64, 16), ("f32", 4, 2, 32, 48), ("f32", 8, 1, 128, 16), ("f32", 2, 1, 256, 32), ("f32", 6, 2, 64, 64),
    ("bf16", 8, 2, 64, 16), ("bf16", 4, 4, 32, 16), ("bf16", 4, 2, 128, 32), ("bf16", 16, 1, 64, 128), ("bf16", 6, 2, 64, 16),
    ("bf16", 2, 1, 256, 64), ("bf16", 4, 1, 128, 256)])
def test_tile_attention_head_dims_pages_and_groups(dtype, n_q, n_kv, hd, page):
    w = workload("tile", dtype, 128, n_q, n_kv, hd, 128, MIX, page=page)
    data = gen.generate(w)
    md = gen.metadata(w)
    # what a cache page holds past its sequence's last position must not be read as a value
    for s, (_, ctx) in enumerate(w.seqs):
        pg = int(md["block_table"][s, (ctx - 1) // page])
        data["v_cache"][0][pg, :, :, (ctx - 1) % page + 1:] = float("nan")
        data["k_cache"][0][pg, :, (ctx - 1) % page + 1:] = float("nan")
    clean = dict(data, k_cache=[torch.nan_to_num(data["k_cache"][0])], v_cache=[torch.nan_to_num(data["v_cache"][0])])
    run = GpuRun(w, data)
    y, k, v = run.run(B.sequential())
    y1, _, _ = run.run(B.nano_schedule(w.nano_rows))
    assert torch.equal(y.view(torch.uint8), y1.view(torch.uint8)), "the split schedule changed bits"
    err = check_against_oracle(w, clean, y, torch.nan_to_num(k), torch.nan_to_num(v))
    say("%s %d/%d x %d, page %d: %.2e" % (dtype, n_q, n_kv, hd, page, err))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_later_tokens_nan_stays_out_of_the_earlier_tokens(dtype):
    """Token 21 of a 40-token prompt is NaN: its key and value are NaN, tokens 0..20 must come out as without it."""
    w = workload("nan", dtype, 128, 4, 2, 64, 128, [(40, 40), (1, 30)])
    data = gen.generate(w)
    y0, _, _ = GpuRun(w, data).run(B.sequential())
    bad = dict(data, x=data["x"].clone())
    bad["x"][21] = float("nan")
    y1, _, _ = GpuRun(w, bad).run(B.sequential())
    keep = list(range(21)) + [40]
    assert torch.isfinite(y1[keep].float()).all()
    assert torch.equal(y0[keep].view(torch.uint8), y1[keep].view(torch.uint8))
    assert torch.isnan(y1[21:40].float()).all()


def test_unaligned_caches_take_the_plain_loops_and_agree():
    w = workload("unaligned", "f32", 128, 4, 2, 64, 128, MIX)
    data = gen.generate(w)
    run = GpuRun(w, data)
    y0, _, _ = run.run(B.sequential())
    step = B.DeviceStep(run.layer, data)
    pools = []
    for c in (step.k_cache, step.v_cache):
        flat = torch.empty(c.numel() + 8, dtype=c.dtype, device=c.device)
        flat[1:1 + c.numel()] = c.reshape(-1)
        pools.append(flat)
    step.batch.k_cache = pools[0].data_ptr() + 4
    step.batch.v_cache = pools[1].data_ptr() + 4
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    run.layer.forward(step.batch, B.sequential(), st)
    torch.cuda.synchronize()
    got, ref = step.y.cpu().double().numpy(), y0.double().numpy()
    assert np.abs(got - ref).max() / np.abs(ref).max() < 1e-5        # two fp32 attention orders


# experts' rows around the edges of the 64-, 128-, 192- and 256-row tile bodies: popular experts with several m tiles, one without rows
@pytest.mark.parametrize("tokens,pull", [(420, 0.0), (470, 3.0), (700, 1.0), (1100, 2.0)])
def test_expert_tiles_follow_the_rows_each_expert_gets(tokens, pull):
    w = workload("wide", "bf16", 512, 4, 1, 128, 512, [(1, 1 + i % 5) for i in range(tokens)], experts=4, top_k=2, seed=50 + tokens)
    data = gen.generate(w)
    router = data["weights"][0]["w_router"]
    router[3] = -router[0]                                   # tokens pulled towards expert 0 never choose expert 3
    x = data["x"].float()
    x += pull * 512 ** 0.5 * router[0] / router[0].norm() * torch.rand(tokens, 1, generator=torch.Generator().manual_seed(1)) ** 0.5
    data["x"] = x.to(torch.bfloat16)
    y, k, v = both_schedules(w, data)
    check_against_oracle(w, data, y, k, v)


# The projection of N columns and depth K: 42 n tiles of 128 (bands of eight, the last of two) with 57, 1, 92 and 97 rows in
# the last m tile; 160 of 128, whole bands; 9 n tiles of 256 (bands of eight and one) with 1 and 57 rows in the last m tile;
# 8 of 256, one whole band
@pytest.mark.parametrize("hidden,inter,rows,N,K,bn,mt", [
    (1024, 2688, 825, 5376, 1024, 128, 128), (1024, 2688, 1025, 5376, 1024, 128, 128), (1024, 2688, 1500, 5376, 1024, 128, 128),
    (1024, 2688, 1537, 5376, 1024, 128, 160), (1280, 10240, 1281, 20480, 1280, 128, 160), (2304, 12288, 1793, 2304, 12288, 256, 128),
    (2304, 12288, 1977, 2304, 12288, 256, 128), (4096, 1024, 2100, 2048, 4096, 256, 128)])
def test_folded_launch_in_bands_matches_smaller_launches(hidden, inter, rows, N, K, bn, mt):
    """Rows of one many-row launch (planes folded, bands over the XCDs, the last band narrower than the others where
    the width is no multiple of it) have the bits of the same rows cut into launches of other tiles, and a
    sample of them, computed alone, is the oracle's."""
    assert (N, K) in ((2 * inter, hidden), (hidden, inter))
    p, few = gemm_path(rows, N, K), gemm_path(40, N, K)
    assert p.folded and p.split > 1 and (p.bn, p.mt) == (bn, mt) and not few.folded
    assert (N // bn) % 8 == {5376: 2, 2304: 1}.get(N, 0)
    w = workload("fold", "bf16", hidden, 4, 1, 128, inter, [(1, 1 + i % 3) for i in range(rows)], seed=60)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, 200, rows))
    data = gen.generate(w)
    y, _, _ = both_schedules(w, data)
    sample = list(range(0, rows, max(rows // 31, 1)))[:31] + [rows - 2, rows - 1]
    sub, d2 = gen.extract_sequences(w, data, sample)
    y2, k2, v2 = GpuRun(sub, d2).run(B.sequential())
    assert torch.equal(y2, y[torch.as_tensor(d2["rows"])])
    check_against_oracle(sub, d2, y2, k2, v2)


def test_projections_of_very_large_weights_walk_n_tiles_in_order():
    """Weights of more than 256 MiB (gate/up 33280 x 8192, down 8192 x 16640): bands of one n tile, on 256 x 256 and on
    128 x 160 tiles.  The bits of the rows in smaller launches, and the oracle's values on a sample."""
    rows, hidden, inter = 1100, 8192, 16640
    p, q = gemm_path(rows, 2 * inter, hidden), gemm_path(rows, hidden, inter)
    assert hidden * inter > 1 << 27 and (p.bn, p.mt, p.kind) == (256, 256, 2) and (q.bn, q.mt, q.kind) == (128, 160, 3)
    w = workload("big", "bf16", hidden, 4, 1, 128, inter, [(1, 1 + i % 3) for i in range(rows)], seed=61)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, 200, rows))
    data = gen.generate(w, device="cuda:0")
    y, _, _ = both_schedules(w, data)
    sub, d2 = gen.extract_sequences(w, data, [0, 255, 256, 511, 700, rows - 1])
    y2, k2, v2 = GpuRun(sub, d2).run(B.sequential())
    assert torch.equal(y2, y[torch.as_tensor(d2["rows"])])
    check_against_oracle(sub, d2, y2, k2, v2)


@pytest.mark.parametrize("rows", [65, 129, 300, 500])
def test_narrow_projections_on_lower_tiles_match_smaller_launches(rows):
    """Outputs so narrow that their (n tile, plane) pairs leave CUs idle take lower tiles; the rows keep the bits they
    have in a 40-row launch."""
    assert all(gemm_path(rows, N, K).kind == 0 and gemm_path(rows, N, K).split > 1 for N, K in ((1536, 1024), (1024, 1024), (4096, 1024), (1024, 2048)))
    w = workload("narrow", "bf16", 1024, 8, 2, 128, 2048, [(1, 1 + i % 7) for i in range(rows)], seed=70)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, 40, rows))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    check_against_oracle(w, data, y, k, v)


def test_work_lists_of_more_rows_than_are_kept_in_registers():
    """4900 rows (the lists' kernel keeps 4096 rows' classification): decodes and two prompts, one past row 4096, with the
    bits of the same rows in smaller dispatches, whether the norm's launch builds the lists or the attention's does."""
    seqs = [(1, 1 + (i * 7) % 600) for i in range(3900)] + [(500, 1300)] + [(1, 1 + i % 40) for i in range(200)] + [(300, 300)]
    w = workload("rows", "bf16", 128, 2, 1, 128, 128, seqs, seed=80)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, 3900, 4400, 4900))
    data = gen.generate(w)
    run = GpuRun(w, data)
    y, _, _ = run.run(B.sequential())
    for merged in ((), (B.DYN_OP_NORM1, B.DYN_OP_QKV, B.DYN_OP_ROPE_KV)):       # lists beside each part's norm; one norm for all, lists by the attention
        y1, _, _ = run.run(B.nano_schedule(w.nano_rows, merged_ops=merged))
        assert torch.equal(y.view(torch.uint8), y1.view(torch.uint8))
    sub, d2 = gen.sub_batch(w, data, [0, 77, 3899, 3900, 3950, len(seqs) - 1])
    y2, k2, v2 = GpuRun(sub, d2).run(B.sequential())
    assert torch.equal(y2, y[torch.as_tensor(d2["rows"])])
    assert torch.isfinite(y.float()).all()


# the general attention kernel keeps 512 scores: chunks of one block, of a block and one position, of several
@pytest.mark.parametrize("dtype,hd,page,chunk", [("f32", 16, 16, 512), ("f32", 16, 16, 1024), ("f32", 8, 24, 2040), ("bf16", 64, 24, 1032)])
def test_general_attention_with_chunks_longer_than_its_scores(dtype, hd, page, chunk):
    w = workload("long_chunk", dtype, 128, 2, 1, hd, 128, [(1, 512), (1, 513), (1, 1025), (3, 1500), (1, 2100), (1, 1)], page=page, seed=90)
    data = gen.generate(w)
    run = GpuRun(w, data, kv_chunk_positions=chunk)
    y, k, v = run.run(B.sequential())
    y1, _, _ = run.run(B.nano_schedule(w.nano_rows))
    assert torch.equal(y.view(torch.uint8), y1.view(torch.uint8))
    say("%s %d %d: %.2e" % (dtype, hd, chunk, check_against_oracle(w, data, y, k, v)))


# planes summed inside the workgroup with 8 X rows a stage (9 rows: 16): 2, 4 and 8 planes of 8 (the fewest there are), 12, 15, 16 and 19 stages.
# `reached` counts the projections of the three that take it on any number of CUs: 8 long planes up to 6 rows, 320 workgroups up to 2
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,inter,rows,reached", [
    (1024, 16, 4, 64, 3072, 1, 3), (1024, 16, 4, 64, 3072, 7, 3), (1024, 16, 4, 64, 3072, 8, 3), (1024, 16, 4, 64, 3072, 9, 0),
    (2048, 16, 4, 128, 7680, 1, 3), (2048, 16, 4, 128, 7680, 6, 3), (2048, 16, 4, 128, 7680, 7, 2), (3072, 24, 8, 128, 8192, 2, 3),
    (3072, 24, 8, 128, 8192, 6, 2), (3072, 24, 8, 128, 8192, 8, 1), (3072, 24, 8, 128, 9728, 1, 3), (3072, 24, 8, 128, 9728, 5, 2),
    (4096, 32, 1, 128, 1024, 2, 3), (4096, 32, 1, 128, 1024, 8, 2)])
def test_few_rows_match_the_bits_of_larger_launches(hidden, n_q, n_kv, hd, inter, rows, reached):
    assert sum(planes_in_workgroup(rows, N, K) for N, K in (((n_q + 2 * n_kv) * hd, hidden), (hidden, n_q * hd), (hidden, inter))) == reached
    w = workload("few_rows", "bf16", hidden, n_q, n_kv, hd, inter, [(1, 1 + (i * 31) % 300) for i in range(21)], seed=95)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, rows, 21))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    check_against_oracle(w, data, y, k, v)


# query blocks of 80 (G = 3), 48 (G = 5), 32 (G = 7) and 16 (G = 11) positions: the first two do not divide a chunk of 1024,
# so the block across position 1024 has tokens without a key in its second chunk
@pytest.mark.parametrize("n_q,n_kv", [(3, 1), (5, 1), (6, 2), (7, 1), (11, 1)])
def test_prompts_across_the_first_chunk_with_blocks_that_do_not_divide_it(n_q, n_kv):
    w = workload("straddle", "bf16", 128, n_q, n_kv, 128, 128, [(1100, 1100), (1, 70), (90, 1060), (3, 1025), (2, 1024), (200, 2150), (1, 1030)], seed=97)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d/%d: %.2e" % (n_q, n_kv, check_against_oracle(w, data, y, k, v)))


# the prompt kernel's chunks (1024 positions, 2048 behind 8192) are shorter than the handle's: 4, 5 and 3 of them for prompts here
@pytest.mark.parametrize("chunk", [1536, 2048, 8192, 65536])
def test_prompts_under_a_handle_with_long_chunks(chunk):
    w = workload("long_handle_chunk", "bf16", 128, 4, 1, 128, 128, [(3100, 3100), (1, 70), (40, 4120), (1, 2049), (2, 8300), (1, 5000), (3, 1025)], seed=98)
    data = gen.generate(w)
    run = GpuRun(w, data, kv_chunk_positions=chunk)
    y, k, v = run.run(B.sequential())
    y1, _, _ = run.run(B.nano_schedule(w.nano_rows))
    assert torch.equal(y.view(torch.uint8), y1.view(torch.uint8)), "the split schedule changed bits"
    say("chunk %d: %.2e" % (chunk, check_against_oracle(w, data, y, k, v)))


@pytest.mark.parametrize("dtype,rows,hd,table_positions", [("bf16", 1030, 32, 131072), ("f32", 1037, 32, 131072), ("f32", 1040, 8, 524288)])
def test_attention_under_a_table_much_wider_than_the_contexts(dtype, rows, hd, table_positions):
    """One q head per kv head and a table so wide that the workgroups of all its chunks (256 threads each, 64 in the
    general form of the 8-wide heads) are more than 2^32 threads: several launches, in the tile form each with
    workgroups past its last row at 1037 rows.  The same bits as under a table as wide as the longest context, and
    as in smaller dispatches."""
    w = workload("wide_table", dtype, 128, 32, 32, hd, 128, [(40, 40)] + [(1, 1 + (7 * i) % 300) for i in range(rows - 42)] + [(1, 1500), (1, 3000)], seed=99)
    data = gen.generate(w)
    y0, k0, v0 = both_schedules(w, data)
    check_against_oracle(w, data, y0, k0, v0)
    table = np.zeros((data["block_table"].shape[0], table_positions // 16), dtype=np.int32)
    table[:, :data["block_table"].shape[1]] = data["block_table"]
    y, k, v = both_schedules(w, dict(data, block_table=table))
    for a, b in ((y, y0), (k, k0), (v, v0)):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
