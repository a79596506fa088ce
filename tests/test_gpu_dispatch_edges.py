"""GPU tests at the edges of dispatch rules: sizes on both sides of a line, against the oracle and against the
same rows in other launches."""
import pytest
import torch

from gpu_util import GpuRun, check_against_oracle, say
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
