"""GPU tests at the edges of dispatch rules: sizes on both sides of a line, against the oracle and against the
same rows in other launches."""
import ctypes

import pytest
import torch

from gpu_util import GpuRun, as_f64, check_against_oracle, gemm_path, row_rel_err, say
from paper_2605_21603_amd import binding as B
from test_gpu_generic_paths import both_schedules, workload
from workloads import gen

pytestmark = pytest.mark.gpu


# Decode attention deals items over workgroups below four rounds of 2048 waves (fewer workgroups when there are
# fewer items): 1 item, 7, 2047 and 2049, and 8184 and 8200 (kv heads x tokens of one chunk each).
@pytest.mark.parametrize("n_kv,tokens", [(1, 1), (1, 7), (23, 89), (3, 683), (12, 682), (8, 1025)])
def test_decode_items_reach_every_token_and_head(n_kv, tokens):
    w = workload("deal", "bf16", 128, n_kv, n_kv, 128, 128, [(1, 1 + (5 * i) % 33) for i in range(tokens)], seed=60 + tokens)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d items: %.2e" % (n_kv * tokens, check_against_oracle(w, data, y, k, v)))


# Attention for other shapes lists its items from 512 workgroups of the dense grid up to 1024 rows: sequentially the first
# batch has 1030 rows (dense) and its second micro-batch 1024 (listed); the others are listed whole and dense or listed in
# parts.  Groups that end in every place of a thread's four rows, sequences of one and several tokens in turn.
@pytest.mark.parametrize("dtype,n_q,n_kv,hd,page,seqs", [
    ("bf16", 4, 2, 64, 16, [(6, 30)] + [(1, 1 + (11 * i) % 300) for i in range(1024)]),
    ("bf16", 6, 2, 64, 16, [(301, 700)] + [(1 + i % 3, 40 + 13 * i) for i in range(60)]),
    ("bf16", 8, 1, 128, 32, [(1, 5000)] + [(1, 1 + 97 * i) for i in range(31)] + [(2, 513)]),
    ("f32", 4, 4, 32, 48, [(1, 1)] + [(5 + i % 13, 20 + 31 * i) for i in range(40)]),
    ("bf16", 2, 1, 256, 64, [(17, 17), (1, 9000), (40, 257), (1, 256), (1, 512), (1, 513), (500, 600)])])
def test_tile_attention_lists_every_item_once(dtype, n_q, n_kv, hd, page, seqs):
    w = workload("list", dtype, 128, n_q, n_kv, hd, 128, seqs, page=page, seed=70 + n_q)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d rows: %.2e" % (w.n_tokens, check_against_oracle(w, data, y, k, v)))


# An infinity among the cached values, in a tile that every column sees whole: its sequence's output rows are NaN (the norm behind the
# attention makes them so, whether the attention gave an infinity or NaN), every other row keeps its bits.
@pytest.mark.parametrize("dtype,hd,page", [("bf16", 64, 16), ("bf16", 128, 32), ("f32", 64, 16)])
def test_an_infinite_cached_value_stays_in_its_sequence(dtype, hd, page):
    w = workload("inf", dtype, 256, 4, 2, hd, 128, [(40, 300), (1, 200), (1, 500), (20, 90), (1, 40)], page=page, seed=78)
    data = gen.generate(w)
    clean, _, _ = both_schedules(w, data)
    rows = torch.arange(w.n_tokens)
    hit = (rows < 40) | (rows == 41)
    for s in (0, 2):
        data["v_cache"][0][data["block_table"][s, 100 // page], 1, 5, 100 % page] = float("inf")
    y, _, _ = both_schedules(w, data)
    assert torch.isnan(y[hit].float()).all()
    assert torch.equal(y[~hit], clean[~hit]) and torch.isfinite(clean.float()).all()


# fp32 projections of whole 64-deep blocks: 16 x 16, 32 x 32 and 64 x 64 tiles and their edges, one and several blocks a chain
# (depths 512, 1024, 2048 and 4608; odd and even counts), widths that fill no 64-, 32- or 16-wide tile; 1030 and 516 are depths of
# the other form.  The second micro-batch takes other tiles than the whole.
@pytest.mark.parametrize("rows,hidden,n_q,n_kv,hd,inter", [
    (3, 512, 4, 2, 64, 1024), (17, 512, 3, 1, 16, 1536), (47, 1024, 4, 2, 64, 2048), (150, 1024, 8, 4, 64, 4608), (65, 2048, 8, 2, 64, 4100),
    (129, 512, 8, 8, 64, 8196), (200, 512, 2, 1, 64, 6148)])
def test_fp32_projections_of_whole_blocks(rows, hidden, n_q, n_kv, hd, inter):
    head = rows // 3
    seqs = ([(head, head)] if head else []) + [(1, 1 + (7 * i) % 40) for i in range(rows - head)]
    w = workload("f32_blocks", "f32", hidden, n_q, n_kv, hd, inter, seqs, seed=80 + rows)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    err = check_against_oracle(w, data, y, k, v)
    say("rows %d: %.2e" % (rows, err))
    assert err < 2e-6                                        # eight chains of K / 8 terms: as in the test of the other tiles


def test_fp32_projections_take_weights_at_any_float():
    """Weights that start 4 bytes off a 16-byte line take loads of single rows where 64 x 64 tiles copy 16 bytes: the same bits."""
    w = workload("f32_off", "f32", 512, 8, 8, 64, 8192, [(200, 200)], seed=90)
    data = gen.generate(w)
    run = GpuRun(w, data)
    y0, _, _ = run.run(B.sequential())
    for n in ("w_qkv", "w_o", "w_gate_up", "w_down"):
        t = run.weights[0][n]
        flat = torch.empty(t.numel() + 4, dtype=t.dtype, device=t.device)
        flat[1:1 + t.numel()] = t.reshape(-1)
        run.weights[0][n] = flat[1:1 + t.numel()].view(t.shape)
    run.layer = B.DynLayer(B.make_config(w.shape, 0), run.weights)
    y1, _, _ = run.run(B.sequential())
    assert torch.equal(y0, y1)


# planes summed inside the workgroup with 16 X rows a stage (6 and 7 rows: 8): 2, 4 and 8 planes of 8, 12, 15, 16, 19 and 28 stages (four on their
# way), up to the last row it is taken for (16; 6 with 257..511 workgroups; two planes of a wide gate/up projection), against the bits of 21 and
# of the remaining rows in other launches
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,inter,rows,reached", [
    (1024, 16, 4, 64, 3072, 9, 3), (1024, 16, 4, 64, 3072, 16, 3), (2048, 16, 4, 128, 7680, 13, 4), (2048, 16, 4, 128, 7680, 16, 4),
    (3072, 24, 8, 128, 8192, 6, 4), (3072, 24, 8, 128, 8192, 7, 3), (3072, 24, 8, 128, 9728, 15, 2), (4096, 32, 1, 128, 14336, 16, 2),
    (2048, 32, 8, 64, 8192, 11, 3)])
def test_up_to_16_rows_match_the_bits_of_larger_launches(hidden, n_q, n_kv, hd, inter, rows, reached):
    wide = B.lib()._ZN3dyn26gemm_rows16_wide_supportedEiiii
    shapes = (((n_q + 2 * n_kv) * hd, hidden), (hidden, n_q * hd), (hidden, inter), (2 * inter, hidden))
    assert sum(wide(rows, N, K, gemm_path(rows, N, K).split) & 0xff != 0 for N, K in shapes) == reached
    w = workload("up_to_16", "bf16", hidden, n_q, n_kv, hd, inter, [(1, 1 + (i * 31) % 300) for i in range(21)], seed=96)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, rows, 21))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    check_against_oracle(w, data, y, k, v)


# The same kernel on a partition of the CUs, which large projections of 5 rows and more and those that a norm follows leave earlier than on the whole
# chip: both forms give the whole chip's bits.
@pytest.mark.parametrize("hidden,inter,rows,on_all,on_part", [
    (4096, 14336, 16, 0b110, 0b000), (4096, 14336, 8, 0b110, 0b010), (4096, 14336, 4, 0b111, 0b111), (3072, 8192, 16, 0b111, 0b111), (3584, 4096, 9, 0b110, 0b100)])
def test_few_rows_on_a_partition(hidden, inter, rows, on_all, on_part):
    taken = B.lib()._ZN3dyn17gemm_rows16_takenEiiiiib
    shapes = ((hidden + 1024, hidden, False), (hidden, hidden, True), (hidden, inter, False))       # qkv, o (its norm follows), down

    def forms(n_cus):
        return sum((taken(rows, N, K, gemm_path(rows, N, K).split, n_cus, norm) & 0xff != 0) << i for i, (N, K, norm) in enumerate(shapes))
    assert forms(0) == forms(256) == on_all and forms(64) == forms(192) == on_part
    w = workload("part_rows", "bf16", hidden, hidden // 128, 4, 128, inter, [(1, 1 + (i * 31) % 300) for i in range(rows)], seed=97)
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    for mask in (0xff, 0xffffff):
        part = run.run(B.nano_schedule([0, rows], chain=B.DENSE_CHAIN, partitions=[1], cu_masks=[[mask] * 8]))
        for a, b in zip(whole, part):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


# The gate applied by the launch that sums a gate/up projection's planes (or, up to 16 rows, reading what the rows' kernel left in the
# plane buffer) gives the bits of the gate as a launch of its own, which stays where a micro-batch folds its planes in registers:
# 2 and 4 planes (4 from a depth of 2048 on), parts of a batch on either side of the folded path.
@pytest.mark.parametrize("hidden,inter,cuts,folded", [
    (1024, 2048, (0, 700, 1300), (True, False, False)), (1024, 2048, (0, 9, 1300), (True, False, True)), (1024, 1984, (0, 5, 21), (False, False, False)),
    (2048, 2048, (0, 17, 150), (False, False, False)), (2048, 2048, (0, 300, 1300), (True, False, True))])
def test_gate_with_the_planes_sum_matches_the_gate_alone(hidden, inter, cuts, folded):
    uses = B.lib()._ZN3dyn22gemm_uses_plane_bufferEiiii
    rows = (cuts[-1], cuts[1], cuts[2] - cuts[1])
    assert tuple(not uses(1, r, 2 * inter, hidden) & 0xff for r in rows) == folded
    seqs = [(1, 1 + (i * 17) % 90) for i in range(cuts[1])] + [(rows[2], rows[2])]
    w = workload("gate", "bf16", hidden, 4, 2, 64, inter, seqs, seed=100 + rows[0])
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, cuts)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)                        # the whole batch and its parts: the same bits
    say("%d rows: %.2e" % (rows[0], check_against_oracle(w, data, y, k, v)))


# Rotary and cache append inside the few rows' qkv projection: heads of 16 to 256, 2 and 4 and 8 planes, 8 and 16 X rows a stage, pages
# of 16 and 48, and a head dim that keeps its own launch (8); the first micro-batch takes the fused form where the whole batch of 21
# rows does not, and gives the same bits in the output and in both caches.
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,page,rows", [
    (1024, 8, 4, 64, 16, 1), (1024, 16, 8, 16, 16, 9), (2048, 8, 2, 32, 48, 16), (2048, 8, 4, 128, 16, 7), (4096, 6, 1, 256, 16, 13), (1024, 8, 4, 8, 16, 5)])
def test_rotary_inside_the_few_rows_projection(hidden, n_q, n_kv, hd, page, rows):
    N = (n_q + 2 * n_kv) * hd
    S = gemm_path(rows, N, hidden).split
    assert S > 1 and B.lib()._ZN3dyn26gemm_rows16_wide_supportedEiiii(rows, N, hidden, S) & 0xff != 0
    w = workload("rows_rope", "bf16", hidden, n_q, n_kv, hd, 1024, [(1, 1 + (i * 131) % 900) for i in range(20)] + [(1, 6000)], page=page, seed=120 + rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, rows, 21))
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    parts = run.run(B.nano_schedule(w.nano_rows, chain=B.DENSE_CHAIN))
    for a, b in zip(whole, parts):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    say("%d rows, heads of %d: %.2e" % (rows, hd, check_against_oracle(w, data, *whole)))


# Expert tiles of at most 64, 128, 192 and 256 rows where an XCD's tiles run at once (4, 16 and 24 n tiles of 256), and of 256 with an expert's
# rows in unequal tiles where they do not (56 n tiles; the second micro-batch has other tiles): no row twice, none left out.
@pytest.mark.parametrize("inter,tokens,pull", [(512, 1000, 1.0), (2048, 600, 0.0), (2048, 1050, 1.5), (3072, 1200, 1.0), (7168, 450, 0.0), (7168, 900, 2.0)])
def test_expert_tiles_in_one_round_and_in_several(inter, tokens, pull):
    w = workload("rounds", "bf16", 256, 2, 1, 128, inter, [(1, 1 + i % 5) for i in range(tokens)], experts=4, top_k=2, seed=140 + tokens)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, tokens // 9, tokens))
    data = gen.generate(w)
    router = data["weights"][0]["w_router"]
    router[2] = -router[0]                                   # tokens pulled towards expert 0 never choose expert 2
    x = data["x"].float()
    x += pull * 256 ** 0.5 * router[0] / router[0].norm() * torch.rand(tokens, 1, generator=torch.Generator().manual_seed(2)) ** 0.5
    data["x"] = x.to(torch.bfloat16)
    y, k, v = both_schedules(w, data)
    say("%d tokens: %.2e" % (tokens, check_against_oracle(w, data, y, k, v)))


# Up to 200 rows per expert on average: 128-wide tiles of 64 to 256 rows by the expert's own count, without planes (512 deep) and with (1024), an
# expert of several tiles, one without rows; 64 tokens, and the smaller micro-batches, on 64-row tiles throughout.
@pytest.mark.parametrize("hidden,tokens,pull", [(512, 64, 0.0), (512, 130, 3.0), (512, 260, 1.0), (1024, 66, 0.0), (1024, 390, 2.0), (1024, 399, 0.5)])
def test_expert_tiles_of_few_rows_follow_the_counts(hidden, tokens, pull):
    w = workload("counts", "bf16", hidden, 4, 1, 128, 512, [(1, 1 + i % 5) for i in range(tokens)], experts=4, top_k=2, seed=90 + tokens)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, tokens // 3, tokens))
    data = gen.generate(w)
    router = data["weights"][0]["w_router"]
    router[2] = -router[0]                                   # tokens pulled towards expert 0 never choose expert 2
    x = data["x"].float()
    x += pull * hidden ** 0.5 * router[0] / router[0].norm() * torch.rand(tokens, 1, generator=torch.Generator().manual_seed(3)) ** 0.5
    data["x"] = x.to(torch.bfloat16)
    y, k, v = both_schedules(w, data)
    say("%d tokens: %.2e" % (tokens, check_against_oracle(w, data, y, k, v)))


# The router in the launch of the second norm, with planes and without: rows of less than one vector per thread, of three and of five, all experts
# but one chosen, counts of experts that are no power of two, 16 experts (a launch of its own).  A workspace a byte too small for that (`apart`) gives the
# router its own launch, with the same bits.
@pytest.mark.parametrize("hidden,experts,top_k,rows,apart", [
    (512, 8, 1, 4, True), (512, 8, 1, 130, False), (4608, 3, 2, 21, False), (8320, 5, 3, 2, False), (8320, 8, 7, 40, False), (256, 8, 2, 600, False), (4096, 16, 2, 30, False)])
def test_router_inside_the_second_norm(hidden, experts, top_k, rows, apart):
    inter = 1024 if hidden == 512 else 128
    w = workload("route", "bf16", hidden, 8, 2, 128, inter, [(1, 1 + i % 5) for i in range(rows)], experts=experts, top_k=top_k, seed=40 + rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, (rows + 2) // 3, rows))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    if apart:
        run = GpuRun(w, data)
        one_stream = B.nano_schedule(w.nano_rows, chain=B.MOE_CHAIN, streams=[0, 0])
        step = B.DeviceStep(run.layer, data, sched=one_stream)
        step.batch.workspace_bytes -= 1
        run.layer.forward(step.batch, one_stream, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert torch.equal(step.y.cpu().view(torch.uint8), y.view(torch.uint8))
    say("%d rows of %d: %.2e" % (rows, hidden, check_against_oracle(w, data, y, k, v)))


# A long prompt's chunks grow with its rows, here from 1024 (2048) to 2048 and 4096 positions: with other sequences around it, in
# another micro-batch than theirs, the same bits; the rows of its end as a step of their own, which keeps the shorter chunks, agree to bf16 rounding.
@pytest.mark.parametrize("prompt,cached", [(4200, 100), (4097, 5003)])
def test_long_prompts_take_longer_chunks(prompt, cached):
    seqs = [(prompt, cached + prompt), (1, 77), (33, 40)]
    w = workload("long", "bf16", 128, 32, 8, 128, 128, seqs, seed=prompt)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    y, end = y[:prompt], 1000
    w_end = workload("end", "bf16", 128, 32, 8, 128, 128, [(end, cached + prompt)])
    rows = slice(prompt - end, prompt)
    part = dict(data, x=data["x"][rows].contiguous(), k_cache=list(k), v_cache=list(v), seq_of_token=data["seq_of_token"][rows],
                pos_of_token=data["pos_of_token"][rows], block_table=data["block_table"][:1], q_start=[0, end], ctx_len=data["ctx_len"][:1])
    y_end = GpuRun(w_end, part).run(B.sequential())[0]
    assert row_rel_err(as_f64(y_end), as_f64(y[-end:])) < 2e-2         # TOL of a bf16 layer
    assert not torch.equal(y_end, y[-end:])                           # the cuts differ


# Prompts behind thousands of positions, each in a micro-batch of its own and all in one dispatch of more rows than that: the same chunks, so the same
# bits - two prompts, one beside decodes, one across position 8192, 1024 rows that begin inside a block of positions; then runs at the 2560 rows
# from which on their length is read off the rows around, and above.
@pytest.mark.parametrize("n_q,n_kv,rows,prompts,cached,decodes", [
    (64, 8, 600, 2, 5000, 0), (64, 8, 1000, 1, 4096, 64), (32, 8, 700, 1, 7900, 400), (128, 8, 1000, 1, 2048, 40), (64, 8, 1024, 1, 5013, 1),
    (64, 8, 2550, 1, 5013, 20), (32, 8, 2560, 1, 7000, 3), (32, 8, 2600, 2, 4090, 0), (40, 8, 2700, 1, 3001, 70)])
def test_prompts_are_cut_alike_in_dispatches_of_any_size(n_q, n_kv, rows, prompts, cached, decodes):
    seqs = [(rows, cached + rows)] * prompts + [(1, 1 + i % 90) for i in range(decodes)]
    w = workload("cuts", "bf16", 128, n_q, n_kv, 128, 128, seqs, seed=cached)
    both_schedules(w, gen.generate(w))


# The merge's forms: one and two chunks four groups of eight heads at a time, up to eight, more, and more than 64 in two levels; head counts that
# leave groups of eight part-filled, dims of one and two loads a lane.
@pytest.mark.parametrize("dtype,n_q,n_kv,hd", [("bf16", 12, 3, 128), ("bf16", 40, 8, 64), ("f32", 3, 1, 64), ("f32", 2, 2, 256), ("bf16", 36, 12, 32)])
def test_merge_of_every_number_of_chunks(dtype, n_q, n_kv, hd):
    seqs = [(1, c) for c in (1, 64, 65, 128, 129, 512, 513, 1100, 4096, 4200)] + [(70, 100), (2, 300)]
    w = workload("merge", dtype, 128, n_q, n_kv, hd, 128, seqs, seed=n_q)
    data = gen.generate(w)
    run = GpuRun(w, data, kv_chunk_positions=64)
    y, k, v = run.run(B.sequential())
    say("%d heads of %d: %.2e" % (n_q, hd, check_against_oracle(w, data, y, k, v)))


# fp32 steps whose projections normalise their rows themselves (256 wide to 32 rows, 768 to 10, 1024 to 8) and gate at any depth, in turn with
# ones that do not (a micro-batch or the batch past the line, 2048 wide): the same bits, over two layers.
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,inter,cut,rows", [
    (256, 4, 4, 64, 1024, 3, 4), (256, 4, 2, 64, 160, 32, 65), (256, 2, 2, 64, 96, 17, 32), (768, 12, 12, 64, 3072, 10, 21), (1024, 16, 4, 64, 512, 8, 17),
    (1024, 8, 2, 128, 64, 1, 8), (512, 8, 8, 32, 1024, 9, 16), (2048, 4, 4, 64, 64, 1, 3), (260, 4, 4, 64, 128, 2, 9)])
def test_fp32_norm_and_gate_inside_the_projections(hidden, n_q, n_kv, hd, inter, cut, rows):
    sh = gen.LayerShape("f32", hidden, n_q, n_kv, hd, inter, n_layers=2)
    w = gen.Workload("norm_in", sh, tuple((1, 1 + (7 * i) % 50) for i in range(rows)), 300 + rows, (0, cut, rows))
    data = gen.generate(w)
    data["x"] = data["x"] * torch.logspace(-3, 3, rows)[:, None]
    y, k, v = both_schedules(w, data)
    err = check_against_oracle(w, data, y, k, v)
    say("%d rows of %d: %.2e" % (rows, hidden, err))
    assert err < 5e-6                                        # two layers of what one layer's test allows


# Decodes beside a prompt in one launch: one query block and one decode, more blocks than half of the workgroups and few, decodes of no
# round and of several; the prompt and the decodes as micro-batches of their own are launches of their own, with the same bits; on a partition of 64 CUs too.
@pytest.mark.parametrize("n_q,n_kv,prompt,cached,n_decode,ctx", [
    (1, 1, 2, 0, 1, 1), (4, 1, 33, 7, 130, 700), (32, 8, 300, 600, 3, 2000), (12, 12, 700, 0, 40, 300), (16, 16, 1500, 0, 9, 4000), (3, 1, 81, 1000, 300, 64)])
def test_decodes_beside_a_prompt(n_q, n_kv, prompt, cached, n_decode, ctx):
    seqs = [(prompt, prompt + cached)] + [(1, 1 + (ctx - 1) * (n_decode - i) // n_decode) for i in range(n_decode)]
    w = workload("mixed", "bf16", 128, n_q, n_kv, 128, 128, seqs, seed=prompt)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    y_part, _, _ = GpuRun(w, data).run(B.nano_schedule([0, w.nano_rows[-1]], chain=B.DENSE_CHAIN, partitions=[1], cu_masks=[[0xff] * 8]))
    assert torch.equal(y.view(torch.uint8), y_part.view(torch.uint8))
    say("%d + %d: %.2e" % (prompt, n_decode, check_against_oracle(w, data, y, k, v)))


# A wide gate/up projection (256 and 383 tiles) of up to 128 rows on the few-row form gives the many-row form's bits (129 rows and more).
@pytest.mark.parametrize("inter,few", [(16384, 1), (24512, 128)])
def test_wide_projections_of_few_rows(inter, few):
    assert [gemm_path(r, 2 * inter, 256).kind for r in (1, 128)] == [0, 0] and gemm_path(400, 2 * inter, 256).kind != 0     # GEMM_FEW
    w = workload("wide_few", "bf16", 256, 2, 1, 128, inter, [(1, 1 + i % 7) for i in range(few + 400)], seed=inter)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, few, few + 400))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d columns: %.2e" % (2 * inter, check_against_oracle(w, data, y, k, v)))


# Gate/up launches cut into tiles of several heights (four 192-row m tiles and one of 64 for 800 rows, ..): every row once, with the bits of the
# smaller launches' tiles; widths whose n tiles fill the bands and do not.
@pytest.mark.parametrize("inter,rows,cut", [(14336, 800, 300), (14336, 1061, 40), (14336, 1300, 700), (14080, 1700, 500), (14336, 2112, 64)])
def test_many_rows_on_tiles_of_several_heights(inter, rows, cut):
    tiles, f = (ctypes.c_int * 4)(), B.lib()._ZN3dyn8wide_cutEiifPNS_7WideCutE
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.c_void_p], ctypes.c_bool
    p = gemm_path(rows, 2 * inter, 256)
    assert p.kind == 2 and f(rows, 2 * inter, (p.workgroups + 255) // 256 + (0.4 if p.tail_rows else 0.0), tiles)      # GEMM_WIDE
    assert 0 <= 64 * sum((i + 1) * n for i, n in enumerate(tiles)) - rows < 64
    w = workload("heights", "bf16", 256, 2, 1, 128, inter, [(1, 1 + i % 5) for i in range(rows)], seed=rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, cut, rows))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d rows, %s: %.2e" % (rows, list(tiles), check_against_oracle(w, data, y, k, v)))


# Folded planes on tiles of two heights (96 + 128, 128 + 160 and 96 rows alone): the heights hold the rows, every row once, the bits of the launches of fewer rows;
# the same on a partition of 64 CUs, which keeps one height.
@pytest.mark.parametrize("hidden,inter,rows,cut,N", [(2048, 2048, 1700, 500, 3072), (2048, 2048, 2112, 700, 3072), (2048, 5120, 2620, 17, 2048), (4096, 4096, 1500, 900, 4096)])
def test_folded_planes_on_tiles_of_two_heights(hidden, inter, rows, cut, N):
    lib, tiles = B.lib(), (ctypes.c_int * 3)()
    f = lib._ZN3dyn8fold_cutERKNS_8GemmPathEiiPNS_7FoldCutE
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p], ctypes.c_bool
    taken = []
    for n, k in ((hidden + 1024, hidden), (hidden, hidden), (hidden, inter)):
        p = gemm_path(rows, n, k)
        if f(ctypes.byref(p), rows, n, tiles):
            taken.append(n)
            assert p.folded and 0 <= 32 * sum((3 + i) * t for i, t in enumerate(tiles)) - rows < 96
    assert N in taken
    w = workload("two_heights", "bf16", hidden, hidden // 128, 4, 128, inter, [(1, 1 + i % 5) for i in range(rows)], seed=rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, cut, rows))
    data = gen.generate(w)
    run = GpuRun(w, data)
    y, k, v = run.run(B.sequential())
    for sched in (B.nano_schedule(w.nano_rows, chain=B.DENSE_CHAIN), B.nano_schedule([0, rows], chain=B.DENSE_CHAIN, partitions=[1], cu_masks=[[0xff] * 8])):
        assert torch.equal(y.view(torch.uint8), run.run(sched)[0].view(torch.uint8))
    say("%d rows: %.2e" % (rows, check_against_oracle(w, data, y, k, v)))


# Gate/up whose planes are folded and gated in one launch (129 to 512 rows; tiles of 64, 128, 192 and 256 rows, with 64 and 108 n tiles): the bits of planes
# summed by a launch (up to 128 rows), in the workgroup (up to 16) and of the many-row form with a gate of its own (513 rows and more).
@pytest.mark.parametrize("hidden,inter,rows,cut,tile", [(1024, 4096, 145, 16, 64), (1024, 4096, 385, 128, 128), (1024, 4096, 700, 400, 128), (2560, 6912, 300, 90, 192),
                                                        (2560, 6912, 513, 512, 256)])
def test_gate_with_planes_folded(hidden, inter, rows, cut, tile):
    taken = B.lib()._ZN3dyn14gate_fold_rowsEiii
    assert gemm_path(300, 2 * inter, hidden).split > 1 and taken(128, 2 * inter, hidden) == taken(513, 2 * inter, hidden) == 0
    assert tile in [taken(r, 2 * inter, hidden) for r in (cut, rows - cut, rows)]
    w = workload("gate_fold", "bf16", hidden, hidden // 128, 4, 128, inter, [(1, 1 + i % 5) for i in range(rows)], seed=rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, cut, rows))
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d rows: %.2e" % (rows, check_against_oracle(w, data, y, k, v)))


# On a partition of 64 CUs the same planes go over the workgroups again (150 and 340 rows) or stay folded (480, on 256-row tiles), on one of 128 they stay folded: the
# bits of the whole chip.
@pytest.mark.parametrize("rows", [150, 340, 480])
def test_gate_with_planes_on_a_partition(rows):
    w = workload("gate_part", "bf16", 2048, 16, 4, 128, 8192, [(1, 1 + i % 5) for i in range(rows)], seed=rows)
    run = GpuRun(w, gen.generate(w))
    y = run.run(B.sequential())[0]
    for cus in (8, 16):
        sched = B.nano_schedule([0, rows], chain=B.DENSE_CHAIN, partitions=[1], cu_masks=[[(1 << cus) - 1] * 8])
        assert torch.equal(y.view(torch.uint8), run.run(sched)[0].view(torch.uint8))


# The same inside the fp32 projection: tiles of any depth (256, 68) and of whole blocks (512, 1024), 16 and 32 rows high, heads of 32, 64 and
# 256, pages of 16 and 48.  Where the batch or one of its parts keeps the launch of its own - more rows (the first two, whose whole batch
# takes 64 x 64 tiles and tiles of any depth), heads of 128 and 16 - it is the same bits.
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,page,rows,cut", [
    (512, 32, 8, 64, 16, 260, 15), (256, 64, 32, 64, 16, 40, 16), (256, 4, 4, 64, 48, 9, 4), (68, 6, 1, 256, 16, 21, 1), (1024, 16, 4, 64, 16, 230, 47),
    (1024, 18, 6, 32, 48, 150, 100), (512, 4, 2, 128, 16, 21, 9), (512, 6, 1, 16, 16, 21, 9)])
def test_rotary_inside_the_fp32_projection(hidden, n_q, n_kv, hd, page, rows, cut):
    seqs = [(1, 1 + (i * 31) % 200) for i in range(cut)] + [(rows - cut, rows + 90)]
    w = workload("f32_rope", "f32", hidden, n_q, n_kv, hd, 256, seqs, page=page, seed=160 + rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, cut, rows))
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    parts = run.run(B.nano_schedule(w.nano_rows, chain=B.DENSE_CHAIN))
    for a, b in zip(whole, parts):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    err = check_against_oracle(w, data, *whole)
    say("%d rows, heads of %d: %.2e" % (rows, hd, err))
    assert err < 2e-6                                        # as the fp32 projections' own tests


# From 512 rows on the v heads of 16 rows are appended together: prompts behind 0, 16, 7 and 33 positions (whole runs and runs across
# pages), single tokens between them, a last group of 3 rows, pages of 16, 32 and 8; both caches against the bits of parts
# below 512 rows.
@pytest.mark.parametrize("dtype,hidden,n_q,n_kv,hd,page", [("bf16", 1024, 8, 2, 128, 16), ("bf16", 512, 4, 4, 64, 32), ("f32", 128, 4, 2, 64, 16), ("bf16", 256, 2, 1, 32, 8)])
def test_v_of_16_rows_is_appended_whole(dtype, hidden, n_q, n_kv, hd, page):
    seqs = [(300, 300), (1, 77), (1, 16), (100, 116), (1, 1), (48, 55), (64, 97), (16, 16), (20, 53)]
    T = sum(q for q, _ in seqs)
    assert T > 512 and T % 16
    w = workload("v16", dtype, hidden, n_q, n_kv, hd, 512, seqs, page=page, seed=180)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, 301, T))
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    parts = run.run(B.nano_schedule(w.nano_rows, chain=B.DENSE_CHAIN))
    for a, b in zip(whole, parts):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    say("%d rows: %.2e" % (T, check_against_oracle(w, data, *whole)))


# Up to 8 rows of whole 64-deep blocks X is loaded straight into MFMA layout, from 9 on by quads that trade: parts of 8 rows and fewer
# beside a whole batch of 9 to 16, plain, gated and rotary forms, one and several blocks a chain: the same bits.
@pytest.mark.parametrize("hidden,n_q,n_kv,hd,inter,cut,rows", [
    (512, 8, 2, 64, 1024, 1, 9), (1024, 16, 4, 64, 2048, 8, 9), (2048, 4, 2, 128, 1536, 8, 16), (1536, 8, 4, 32, 4608, 3, 11)])
def test_fp32_x_of_few_rows_goes_straight(hidden, n_q, n_kv, hd, inter, cut, rows):
    w = workload("f32_x", "f32", hidden, n_q, n_kv, hd, inter, [(1, 1 + (i * 37) % 120) for i in range(rows)], seed=170 + rows)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, cut, rows))
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    parts = run.run(B.nano_schedule(w.nano_rows, chain=B.DENSE_CHAIN))
    for a, b in zip(whole, parts):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    err = check_against_oracle(w, data, *whole)
    say("%d + %d rows: %.2e" % (cut, rows - cut, err))
    assert err < 2e-6                                        # as the fp32 projections' own tests


def rows_in_runs(seqs):
    """Rows that belong to 16 rows of one sequence at consecutive positions from a multiple of 16 on."""
    return sum(max(0, c // 16 - (c - q + 15) // 16) * 16 for q, c in seqs)


# The runs themselves: a cached prefix that fills its pages or not (runs at slot 0 and at slot 16 of a later page), prompts that
# start on a row that is a multiple of 16 or behind single tokens, sequences that are one run, a run and a rest on either side, or
# just none; pages that hold no whole run.  Parts below 512 rows append row by row: the same bits.
@pytest.mark.parametrize("dtype,page,seqs,runs", [
    ("bf16", 16, [(320, 368), (208, 208)], 528), ("bf16", 32, [(320, 368), (208, 1209)], 512), ("bf16", 64, [(1, 77)] * 3 + [(320, 361), (200, 200)], 496),
    ("f32", 16, [(1, 9)] + [(15 + i % 18, 15 + i % 18 + (7 * i) % 40) for i in range(24)], None), ("f32", 48, [(1, 5)] * 7 + [(16, 32), (17, 32), (31, 47), (30, 45), (500, 517)], 544),
    ("bf16", 24, [(500, 500), (33, 70)], 0), ("f32", 16, [(1, 1 + i % 50) for i in range(400)] + [(140, 150)], 128)])
def test_v_runs_start_anywhere(dtype, page, seqs, runs):
    T = sum(q for q, _ in seqs)
    assert T >= 512 and (runs is None or (rows_in_runs(seqs) if page % 16 == 0 else 0) == runs)
    w = workload("v_runs", dtype, 256, 4, 2, 64, 512, seqs, page=page, seed=190 + T)
    cut = next(sum(q for q, _ in seqs[:i]) for i in range(len(seqs), 0, -1) if sum(q for q, _ in seqs[:i]) < 512)
    w = gen.Workload(w.name, w.shape, w.seqs, w.seed, (0, cut, T))
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    parts = run.run(B.nano_schedule(w.nano_rows, chain=B.DENSE_CHAIN))
    for a, b in zip(whole, parts):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    say("%d rows: %.2e" % (T, check_against_oracle(w, data, *whole)))


def test_v_cache_off_a_16_byte_line_is_appended_row_by_row():
    w = workload("v_off", "f32", 128, 4, 2, 64, 256, [(500, 500), (30, 60)], seed=199)
    data = gen.generate(w)
    run = GpuRun(w, data)
    whole = run.run(B.sequential())
    step = B.DeviceStep(run.layer, data)
    flat = torch.empty(step.v_cache.numel() + 4, dtype=step.v_cache.dtype, device="cuda:0")
    off = flat[1:1 + step.v_cache.numel()].view(step.v_cache.shape)
    off.copy_(step.v_cache)
    step.batch.v_cache = off.data_ptr()
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    run.layer.forward(step.batch, B.sequential(), st)
    st.synchronize()
    assert torch.equal(off.cpu(), whole[2]) and torch.equal(step.k_cache.cpu(), whole[1])


# Layers over lists of 1 pair, a wave's 64 and one more and 1026 of 16 experts (scanned), 1024 of 8 and more than the 8192 pairs of one pass (by sixteen waves).
@pytest.mark.parametrize("tokens,experts,top_k", [(1, 3, 1), (64, 16, 1), (65, 5, 1), (512, 8, 2), (513, 16, 2), (4300, 4, 2)])
def test_expert_lists_hold_every_pair_in_order(tokens, experts, top_k):
    seqs = [(tokens - 1, tokens - 1), (1, 9)] if tokens > 1 else [(1, 9)]
    w = workload("lists", "bf16", 128, 1, 1, 128, 128, seqs, experts=experts, top_k=top_k, seed=200 + tokens)
    data = gen.generate(w)
    y, k, v = both_schedules(w, data)
    say("%d pairs, %d experts: %.2e" % (tokens * top_k, experts, check_against_oracle(w, data, y, k, v)))


# The lists themselves, read back: both sides of the line between the scan and the sixteen waves (512 pairs; 100 an expert from 6 experts on),
# steps of 512 and of 1024 pairs and one more or less, waves without a pair, several passes, pairs that begin past 0, an expert nobody chose.
@pytest.mark.parametrize("experts,n_pairs,scan", [
    (3, 1, 1), (8, 64, 1), (4, 512, 1), (4, 513, 0), (1, 960, 0), (2, 1024, 0), (2, 1025, 0), (8, 800, 1), (8, 801, 0), (16, 513, 1), (16, 1600, 1),
    (16, 1601, 0), (5, 2048, 0), (8, 8192, 0), (8, 8193, 0), (16, 16390, 0)])
def test_expert_lists_read_back(experts, n_pairs, scan):
    lib = B.lib()
    assert lib._ZN3dyn17expert_lists_scanEii(n_pairs, experts) & 0xff == scan
    f = lib._ZN3dyn19launch_expert_listsEPKiiiiiPiS2_P12ihipStream_t
    f.argtypes, f.restype = [ctypes.c_void_p] + [ctypes.c_int] * 4 + [ctypes.c_void_p] * 3, ctypes.c_int
    base, cap = 37, n_pairs + 5
    sel = torch.randint(0, experts, (base + n_pairs,), dtype=torch.int32, generator=torch.Generator().manual_seed(n_pairs))
    if experts > 2:
        sel[sel == 1] = 0
    d_sel, counts, lists = sel.cuda(), torch.full((experts,), -1, dtype=torch.int32, device="cuda:0"), torch.full((experts, cap), -1, dtype=torch.int32, device="cuda:0")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert f(d_sel.data_ptr(), n_pairs, base, experts, cap, counts.data_ptr(), lists.data_ptr(), st.cuda_stream) == 0
    st.synchronize()
    for e in range(experts):
        want = (sel[base:] == e).nonzero().flatten().int() + base
        assert counts[e].item() == len(want)
        assert torch.equal(lists[e, :len(want)].cpu(), want) and (lists[e, len(want):] == -1).all()
