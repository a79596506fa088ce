"""Which work item of the block attention kernels writes which token (no GPU).

The kernels ask column_end (csrc/common.h) what an item does with each of its columns.  Here the rule is compiled for
the host and walked over every (block, chunk) item of a prompt: a token whose keys fit one chunk has its output written
by exactly one item, any other token has exactly one partial per chunk it reaches, and nothing else is written.  The bound on a token's chunks that sizes the partials
(prefill_max_chunks) is walked too, and so is the rule that picks a block's chunk size (prompt_chunk_positions): it depends on
what its own sequence has in the step and on nothing else of the dispatch.  Last, the share of a mixed launch (mixed_share)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

WALK = r"""
#include <cstdio>
#include <vector>
#include "common.h"
using namespace dyn;
// Tokens p0 .. p1 - 1 of one sequence in aligned blocks of `tg` positions; a block's chunk size is chunk_of(block),
// its items are the chunks its last token reaches (kernels_attn_plan.hip, attn_tile_kernel).
template <class F> static long wrong(int p0, int p1, int tg, F chunk_of) {
    std::vector<int> done(p1, 0), partial(p1, 0), chunk(p1, 0);
    for (int p = p0; p < p1;) {
        const int end = p + tg - p % tg < p1 ? p + tg - p % tg : p1, ct = chunk_of((p / tg + 1) * tg);
        for (int c = 0; c * ct < end; ++c)
            for (int t = p; t < end; ++t) {
                chunk[t] = ct;
                const ColumnEnd e = column_end(t + 1, c * ct, ct);
                done[t] += e == COLUMN_DONE;
                partial[t] += e == COLUMN_PARTIAL;
            }
        p = end;
    }
    long bad = 0;
    for (int t = p0; t < p1; ++t) {
        const int chunks = (t + chunk[t]) / chunk[t];
        bad += done[t] != (chunks == 1) || partial[t] != (chunks == 1 ? 0 : chunks);
    }
    return bad;
}
int main() {
    long bad = 0;
    for (int G = 1; G <= 16; ++G) {
        const int TG = 16 / G;
        for (int p0 : {0, 1, 959, 1000}) {
            bad += wrong(p0, 20000, 16 * TG, [](int reach) { return prefill_chunk_positions(reach); });
            for (int rows : {2624, 5120}) bad += wrong(p0, 20000, 16 * TG, [=](int reach) { return prefill_run_chunk_positions(reach, 16 * TG, 8, rows, reach); });
            for (int ct : {64, 240, 256, 1024}) bad += wrong(p0, 3000, 4 * TG, [ct](int) { return ct; });
        }
    }
    // the bound that sizes partials and lists holds for every key count and block, and is met
    for (int G : {1, 3, 4, 16}) {
        const int tg = 16 * (16 / G);
        int most = 1;
        for (int n = 1; n <= 200000; ++n) {
            const int ct = prefill_chunk_positions(((n - 1) / tg + 1) * tg);
            if ((n + ct - 1) / ct > most) most = (n + ct - 1) / ct;
            bad += prefill_max_chunks(n) < most;
            if (n % 65536 == 0 || n % 65536 == 1025) bad += prefill_max_chunks(n) != most;
        }
    }
    for (int nk : {0, -1}) bad += column_end(nk, 0, 64) != COLUMN_NOT_MINE;      // dead columns
    printf("%ld\n", bad);
}
"""


RULE = r"""
#include <cstdio>
#include <vector>
#include "common.h"
using namespace dyn;
// The chunk of every token of a prompt of `n` rows from position p0 on, with `before` and `after` rows of other sequences around it, the run's ends
// looked for from each row as a wave does it from its first and last.
static std::vector<int> chunks(int n, int p0, int before, int after, int tg, int n_kv, long &ends) {
    std::vector<int32_t> seq(before + n + after);
    for (int i = 0; i < (int)seq.size(); ++i) seq[i] = i < before ? i : i < before + n ? before : i - n + 1;
    std::vector<int> out(n);
    for (int i = 0; i < n; ++i) {
        auto count = [&](int row, int step) {
            int k = 0;
            for (int r = row + step; k < 64 && r >= 0 && r < (int)seq.size() && seq[r] == before; r += step) ++k;
            return k;
        };
        const int t = before + i;
        const Run run = run_around(t, (int)seq.size(), count);
        ends += run.start != before || run.end != before + n;
        out[i] = prompt_chunk_positions(t, p0 + i, run.start, run.end, tg, n_kv);
    }
    return out;
}
int main() {
    long other_rows = 0, in_block = 0, short_runs = 0, grown = 0, ends = 0;
    const int heads[][2] = {{32, 8}, {64, 8}, {96, 8}, {128, 8}, {40, 8}, {40, 40}, {12, 12}, {15, 1}};
    for (auto &h : heads) {
        const int tg = 16 * (16 / (h[0] / h[1]));
        for (int n : {2, 40, 600, 1000, 1024, 1025, 2048, 2500, 2559, 2560, 2561, 2600, 2700, 3000, 4096, 9000})
            for (int p0 : {0, 7, 1500, 4096, 5003, 7900, 16300, 32700}) {
                const std::vector<int> alone = chunks(n, p0, 0, 0, tg, h[1], ends);
                for (int i = 0; i < n; ++i) {
                    const int plain = prefill_chunk_positions(((p0 + i) / tg + 1) * tg);
                    in_block += i && (p0 + i) % tg && alone[i] != alone[i - 1];
                    short_runs += n <= kLongRun && alone[i] != plain;
                    grown += alone[i] > plain;
                }
                for (int before : {0, 1, 64, 1100, 2500, 5000})
                    for (int after : {0, 1, 64, 1100, 2500, 5000}) other_rows += chunks(n, p0, before, after, tg, h[1], ends) != alone;
            }
    }
    long uneven = 0;
    for (int ct : chunks(4096, 8192, 1, 1, 64, 8, ends)) uneven += ct != 4096;
    for (int n : {5000, 20000, 100000}) chunks(n, 0, 5, 9, 64, 8, ends);
    printf("%ld %ld %ld %ld %d %ld\n", ends, other_rows, in_block, short_runs, grown > 0, uneven);
}
"""


def compiled(tmp_path, name, source):
    if not os.path.exists(HIPCC):
        pytest.skip("no ROCm toolchain")
    src, exe = tmp_path / (name + ".cpp"), tmp_path / name
    src.write_text(source)
    subprocess.check_call([HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_2605_21603_amd", "csrc"),
                           str(src), "-o", str(exe)], stderr=subprocess.DEVNULL)
    return subprocess.check_output([str(exe)], text=True)


def test_a_prompts_chunks_do_not_depend_on_the_rows_around_it(tmp_path):
    """Alone in its dispatch or with up to 10000 rows around it, on either side, a prompt is cut alike; the tokens of a block are; and a run of
    at most 2560 rows, wherever it begins in its blocks, has the plain rule.  Long prompts' chunks do grow, alike over the whole of one of 4096 rows
behind 8192 positions."""
    assert compiled(tmp_path, "rule", RULE).split() == ["0", "0", "0", "0", "1", "0"]


def test_every_token_is_written_once_whatever_the_block_and_chunk(tmp_path):
    assert int(compiled(tmp_path, "walk", WALK)) == 0


SHARE = r"""
#include <cstdio>
#include "common.h"
using namespace dyn;
int main() {
    long over = 0, outside = 0, full = 0, longer = 0;
    for (int groups : {1, 2, 7, 8, 9, 16, 64, 128, 256})
        for (int items = 1; items < 3000; items += 1 + items / 40)
            for (int parts = 0; parts <= 200; ++parts) {
                const float prompts = items * 40.f, decodes = prompts * parts / 20.f, share = groups * prompts / (prompts + decodes);
                const int n = mixed_share(items, prompts, decodes, groups), least = groups / 2 < 8 ? groups / 2 : 8;
                outside += n < 0 || (groups > 1 && n >= groups);                                 // someone starts on the decodes
                over += items > groups / 4 && n > least && n > (int)(share + 7.001f) / 8 * 8;    // no more than the share, in eights
                longer += items <= groups / 4 && n > 8 && n < items && (items + n - 1) / n > 0.2f * decodes * items / (prompts * groups) + 1;
                full += groups == 256 && parts && items > 64 && n > 0.8f * groups && decodes > 0.3f * prompts;
            }
    printf("%ld %ld %ld %ld %d %d %d %d\n", outside, over, full, longer, mixed_share(288, 702.f, 213.f, 256), mixed_share(384, 3528.f, 3408.f, 256),
           mixed_share(40, 90.f, 500.f, 256), mixed_share(32, 6.f, 8400.f, 256));
}
"""


def test_a_mixed_launch_leaves_the_decodes_their_share(tmp_path):
    """Prompts never start on more workgroups than their part of the estimated work, rounded up to eight (one for each XCD), whatever number of
    rounds that makes; 288 blocks of a share of 196 workgroups go in two rounds of 144, 384 of one of 130 in three.  A few blocks have a workgroup
each, unless that takes workgroups for nothing from decodes that last much longer: 40 beside as much again, 32 beside a thousand times their time."""
    assert compiled(tmp_path, "share", SHARE).split() == ["0", "0", "0", "0", "144", "128", "40", "8"]
