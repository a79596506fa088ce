"""Distance between matrix products and what reads their results, where assembly stands on one side (no GPU).

A vector instruction that touches the destination of a matrix instruction too early reads the old value: the hardware
does not hold it back, the compiler puts the wait states between.  It does so for instructions it issued itself.
Inline assembly it does not look into - a product written as assembly has no latency in its eyes, and an operand of
assembly no hazard.  This replays the compiled kernels: along every path of the control flow, an instruction that
reads or overwrites a product's register must come at least WAIT_STATES later if the product or the instruction is
assembly.  Exempt are the accumulator of a following product, which the hardware forwards, and the destination of an LDS
read, whose data arrive long after.  Only the s_nop that the source itself writes count: what else stands
between in today's build the compiler may move.  The mask that separates the two on some paths is the compiler's
instruction, and a register it has written is no product's any more.  A product written as assembly must not
follow a vector instruction that writes one of its operands within OPERAND_STATES instructions."""
import re

import pytest
from test_isa_host import compile_to_isa, registers

# A 16x16x32 bf16 product is at most an 8-pass instruction: the ISA's table asks 11 wait states before a vector
# instruction touches its result, one more than that covers this generation's longer pipeline.
WAIT_STATES = 12
# and a product that reads what a vector instruction wrote needs two (the compiler sees to its own)
OPERAND_STATES = 2


def parse(body):
    """[(label or None, text, is_asm)] of a kernel's lines."""
    out, asm = [], False
    for x in body:
        s = x.split(";", 1)[0].strip() if not x.strip().startswith(";;#") else x.strip()
        if "ASMSTART" in x:
            asm = True
        elif "ASMEND" in x:
            asm = False
        elif s.endswith(":"):
            out.append((s[:-1], None, False))
        elif s and s[0] not in ".;":
            out.append((None, s, asm))
    return out


def states_of(s, asm):
    m = re.match(r"s_nop (\d+)", s)
    return int(m.group(1)) + 1 if m and asm else 0


def product_read_hazards(body):
    """Instructions that touch a product's destination too early, over all paths."""
    items = parse(body)
    at = {lab: i for i, (lab, _, _) in enumerate(items) if lab}
    entry = {0: {}}                      # item index -> {register: (wait states since the product, product is assembly)} on entry
    work, found = [0], set()
    while work:
        i = work.pop()
        state = dict(entry[i])
        first = True
        while i < len(items):
            label, s, asm = items[i]
            if label and not first:
                break                                              # falls through into a block of its own
            first = False
            if label:
                i += 1
                continue
            op, _, rest = s.partition(" ")
            dst, _, ops = rest.partition(",")
            own = registers(dst) if op.startswith(("v_", "ds_read")) else set()
            if op.startswith("v_mfma"):
                parts = re.findall(r"v\[\d+:\d+\]|v\d+|[^,\s]+", ops)
                sources = registers(" ".join(parts[:2])) | (registers(" ".join(parts[2:3])) - own)
            else:
                sources = registers(ops if op.startswith("ds_read") else rest)
            for r in sources:
                if r in state and state[r][0] < WAIT_STATES and (asm or state[r][1]):
                    found.add((i, s))
            if asm and op.startswith("v_mfma") and any(("w", r) in state for r in registers(rest)):
                found.add((i, s))
            n = states_of(s, asm)
            products = {r: (t + n, a) for r, (t, a) in state.items() if isinstance(r, int) and t + n < WAIT_STATES and r not in own}
            m = max(n, states_of(s, True) if op == "s_nop" else 1)                   # any instruction is a state here
            state = {k: (t + m, a) for k, (t, a) in state.items() if not isinstance(k, int) and t + m < OPERAND_STATES}
            state.update(products)
            for r in own:
                if op.startswith("v_mfma"):
                    state[r] = (0, asm)
                    state.pop(("w", r), None)
                elif op.startswith("v_"):
                    state["w", r] = (0, asm)
            if op.startswith("s_cbranch") or op == "s_branch":
                target = at[rest.strip()]
                merge(entry, target, state, work)
                if op == "s_branch":
                    i = len(items)
                    break
            if op == "s_endpgm":
                i = len(items)
                break
            i += 1
        if i < len(items):
            merge(entry, i, state, work)
    return [s for _, s in sorted(found)]


def merge(entry, i, state, work):
    have = entry.get(i)
    if have is None:
        entry[i] = dict(state)
        work.append(i)
        return
    changed = False
    for r, (t, a) in state.items():
        old = have.get(r)
        new = (t, a) if old is None else (min(t, old[0]), a or old[1])
        if new != old:
            have[r] = new
            changed = True
    if changed:
        work.append(i)


def kernels(lines):
    starts = [i for i, l in enumerate(lines) if re.match(r"^_ZN3dyn\S*kernel\S*:", l)]
    for n, i in enumerate(starts):
        end = starts[n + 1] if n + 1 < len(starts) else len(lines)
        body = lines[i + 1:end]
        stop = [j for j, x in enumerate(body) if ".end_amdhsa_kernel" in x or x.strip().startswith(".section")]
        yield lines[i].split(":")[0], body[:stop[0]] if stop else body


@pytest.mark.parametrize("source", ["kernels_attn_prefill.hip", "kernels_gemm.hip", "kernels_gemm_wide.hip"])
def test_nothing_reads_a_product_before_it_has_left_the_matrix_core(tmp_path, source):
    checked = 0
    for name, body in kernels(compile_to_isa(tmp_path, source)):
        if not any("v_mfma" in x for x in body):
            continue
        assert not product_read_hazards(body), (name, product_read_hazards(body)[:5])
        checked += 1
    assert checked >= 1


def test_the_replay_convicts_a_reader_that_comes_too_early():
    product = "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]"
    asm = lambda s: ["\t;;#ASMSTART", s, "\t;;#ASMEND"]
    read = "\tv_max3_f32 v20, v0, v21, v22"
    nop = lambda n: asm("\ts_nop %d" % n)
    assert product_read_hazards([product] + asm(read)) != []
    assert product_read_hazards([product] + nop(10) + asm(read)) != []
    assert product_read_hazards([product] + nop(11) + asm(read)) == []
    assert product_read_hazards([product, "\ts_nop 15"] + ["\ts_mov_b32 s0, s1"] * 20 + asm(read)) != []   # the compiler's, free to move
    assert product_read_hazards([product, read]) == []                              # both the compiler's: its own wait states
    assert product_read_hazards([product, "\tv_cndmask_b32_e32 v0, v30, v0, vcc"] + asm(read)) == []          # a masked value
    assert product_read_hazards(asm(product) + ["\tv_add_f32_e32 v20, v0, v21"]) != []
    assert product_read_hazards(asm(product) + asm(product)) == []                   # accumulation is forwarded
    write = "\tv_mov_b32_e32 v1, 0"
    assert product_read_hazards([write] + asm(product)) != []
    assert product_read_hazards([write] + nop(0) + asm(product)) != []
    assert product_read_hazards([write] + nop(1) + asm(product)) == []
    assert product_read_hazards([write, product]) == []                             # the compiler's own
    # the distance of the shorter way round a branch counts
    skip = [product, "\ts_cbranch_scc1 .LBB0_2"] + nop(15) + [".LBB0_2:"] + asm(read)
    assert product_read_hazards(skip) != []
    # and the way back to a loop's head
    loop = [".LBB0_1:"] + asm(read) + nop(15) + [product, "\ts_cbranch_scc1 .LBB0_1", "\ts_endpgm"]
    assert product_read_hazards(loop) != []


def touched_in_flight(body):
    """Instructions that name a register of an assembly LDS read before a wait has retired it, over all paths, behind
    the loops that issue such reads as well as in them: a read nobody uses still writes its register when it arrives.
    In state: LDS operations issued since the read (LDS operations retire in order; scalar loads may overtake them
    and retire nothing)."""
    items = parse(body)
    at = {lab: i for i, (lab, _, _) in enumerate(items) if lab}
    entry, work, found = {0: {}}, [0], set()

    def join(i, state):
        have = entry.get(i)
        if have is None:
            entry[i] = dict(state)
            work.append(i)
            return
        new = {r: min(n, have.get(r, n)) for r, n in state.items()}
        if any(have.get(r) != n for r, n in new.items()):
            have.update(new)
            work.append(i)

    while work:
        i = work.pop()
        state, first = dict(entry[i]), True
        while i < len(items):
            label, s, asm = items[i]
            if label:
                if not first:
                    join(i, state)
                    break
                i, first = i + 1, False
                continue
            first = False
            op, _, rest = s.partition(" ")
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", rest)
                if m:
                    state = {r: n for r, n in state.items() if n < int(m.group(1))}
            else:
                if registers(rest) & set(state):
                    found.add((i, s))
                if op.startswith("ds_"):
                    state = {r: n + 1 for r, n in state.items()}
                    if asm and op.startswith("ds_read"):
                        state.update({r: 0 for r in registers(rest.partition(",")[0])})
                if op.startswith("s_cbranch") or op == "s_branch":
                    join(at[rest.strip()], state)
                if op in ("s_branch", "s_endpgm"):
                    break
            i += 1
    return [s for _, s in sorted(found)]


@pytest.mark.parametrize("source", ["kernels_attn_prefill.hip", "kernels_gemm.hip", "kernels_gemm_wide.hip"])
def test_no_register_is_touched_while_a_read_into_it_is_in_flight(tmp_path, source):
    checked = 0
    for name, body in kernels(compile_to_isa(tmp_path, source)):
        if any("ASMSTART" in a and "ds_read" in b for a, b in zip(body, body[1:])):
            assert not touched_in_flight(body), (name, touched_in_flight(body)[:5])
            checked += 1
    assert checked >= 1


def test_the_flight_replay_convicts_a_register_reused_before_its_wait():
    asm = lambda s: ["\t;;#ASMSTART", s, "\t;;#ASMEND"]
    head = [".LBB0_1:", "\ts_waitcnt lgkmcnt(0)"] + asm("\tds_read_b128 v[0:3], v40") + asm("\tds_read_b128 v[4:7], v40 offset:0x800") + ["\ts_cbranch_scc1 .LBB0_1"]
    assert touched_in_flight(head + ["\tv_add_u32_e32 v1, s0, v50", "\ts_waitcnt lgkmcnt(0)"]) != []         # an address where data will land
    assert touched_in_flight(head + ["\ts_waitcnt lgkmcnt(0)", "\tv_add_u32_e32 v1, s0, v50"]) == []
    assert touched_in_flight(head + ["\ts_waitcnt lgkmcnt(1)", "\tv_add_u32_e32 v1, s0, v50"]) == []         # the first read has retired
    assert touched_in_flight(head + ["\ts_waitcnt lgkmcnt(1)", "\tv_add_u32_e32 v5, s0, v50"]) != []
    assert touched_in_flight(head + ["\ts_load_dword s4, s[2:3], 0x0", "\ts_waitcnt lgkmcnt(2)", "\tv_add_u32_e32 v1, s0, v50"]) != []
