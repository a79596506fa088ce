"""The LDS-counter replay of test_isa_host.py over the loops of kernels_gemm_wide.hip (no GPU)."""
from collections import Counter

import pytest
from test_isa_host import MFMA, compile_to_isa, instructions, replay_lds_counter


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    return compile_to_isa(tmp_path_factory.mktemp("isa_wide"), "kernels_gemm_wide.hip")


def hand_laid_loops(body):
    """Every loop that holds assembly MFMAs: from its head to the first branch behind the last one and the reads that follow it."""
    heads = [j for j, x in enumerate(body) if "Loop Header" in x] + [len(body)]
    loops = []
    for a, b in zip(heads, heads[1:]):
        asm = [j for j in range(a, b) if MFMA in body[j] and "ASMSTART" in body[j - 1]]
        if asm:
            last = max(j for j in range(a, min(asm[-1] + 12, b)) if "ASMEND" in body[j] and (MFMA in body[j - 1] or "ds_read" in body[j - 1]))
            loops.append(body[a:last + 1])
    return loops


@pytest.mark.parametrize("kernel,tiles", [("gemm_fold_kernel", [(256, 128)]),
                                          ("gemm_experts_wide_kernelILb0E", [(256, 256), (256, 192), (256, 128), (256, 64)]),
                                          ("gemm_experts_wide_kernelILb1E", [(256, 256), (256, 192), (256, 128), (256, 64)]),
                                          ("gemm_cut_kernelILb0E", [(256, 256), (256, 192), (256, 128), (256, 64)]),
                                          ("gemm_cut_kernelILb1E", [(256, 256), (256, 192), (256, 128), (256, 64)]),
                                          ("gemm_experts_kernelILb0ELb0E", [(128, 256)]), ("gemm_experts_kernelILb1ELb0E", [(128, 256)])])
def test_wide_loops_touch_no_operand_before_its_wait(lines, kernel, tiles):
    starts = [i for i, l in enumerate(lines) if l.startswith("_ZN3dyn") and l.split(";")[0].strip().endswith(":")]
    at = next(i for i in starts if kernel in lines[i])
    body = lines[at:min([s for s in starts if s > at] + [len(lines)])]
    loops = hand_laid_loops(body)
    want = Counter()
    for bn, mt in tiles:                                  # eight waves, two along the X rows; four on a tile taller than wide
        na, nb = (bn // 4 // 16, mt // 32) if bn >= mt else (bn // 2 // 16, mt // 64)
        want[(2 * na * nb, 2 * (na + nb))] += 1
    got = Counter()
    for loop in loops:
        c = Counter(x.split()[0] for x in instructions(loop))
        copies = {k: v for k, v in c.items() if k.startswith(("v_mov", "v_accvgpr", "scratch_", "v_swap", "v_readlane", "v_writelane"))}
        assert not copies, copies
        violations, n_reads = replay_lds_counter(loop)
        assert not violations, violations[:5]
        assert c["s_barrier"] == 1 and n_reads == c["ds_read_b128"]
        got[(c[MFMA], n_reads)] += 1
    assert got == want
