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
