"""Wait states around the asm statements, on the kernels' gfx950 assembly.

The compiler inserts the wait states that the hardware does not interlock, but
only between instructions of its own: what an asm statement holds, and the
instructions just before it, are outside its checks.  The direct loads into
LDS and the MFMAs of the GEMM's 4-wave loop are such statements:

  * a load into LDS reads m0, and needs one wait state after a scalar
    instruction has written it;
  * a buffer or global access needs five wait states after a vector
    instruction (v_readfirstlane, a compare, a spill's v_readlane) has written
    a scalar register that it reads, here a word of the buffer descriptor.  A
    load with an old range would drop rows, or read past the matrix;
  * an MFMA needs two wait states after a vector instruction has written one of
    its operands (the compiler keeps them around MFMAs of its own).

An instruction counts as one wait state, `s_nop n` as n + 1; distances are
taken over every control-flow path.
"""

import collections
import re

import pytest

from conftest import device_asm

SOURCES = ["gemm_f16.hip", "attn_fwd.hip", "attn_bwd.hip"]


def functions(lines):
    """name -> {label: [instructions]} in program order"""
    out, blocks = {}, None
    for line in lines:
        m = re.match(r"^(_Z\S+):", line)
        if m:
            blocks = out[m.group(1)] = collections.OrderedDict(entry=[])
            cur = "entry"
            continue
        if blocks is None:
            continue
        if line.startswith(".Lfunc_end"):
            blocks = None
            continue
        m = re.match(r"^(\.LBB\d+_\d+):", line)
        if m:
            cur = m.group(1)
            blocks[cur] = []
            continue
        t = line.split(";")[0].strip()
        if t and not t.startswith((".", "#")):
            blocks[cur].append(t)
    return out


def predecessors(blocks):
    pred, names = collections.defaultdict(list), list(blocks)
    for k, b in enumerate(names):
        ins = blocks[b]
        succ = [t.split()[1] for t in ins if t.startswith(("s_cbranch", "s_branch"))]
        if not (ins and ins[-1].startswith(("s_branch", "s_endpgm", "s_setpc"))) and k + 1 < len(names):
            succ.append(names[k + 1])
        for s in succ:
            pred[s].append(b)
    return pred


def waits_since(blocks, pred, label, index, need, hit):
    """Fewest wait states between instruction (label, index) and an earlier one
    that `hit` accepts, over all paths; None if there are `need` or more."""
    work, best, seen = [(label, index - 1, 0)], None, {}
    while work:
        b, j, w = work.pop()
        while j >= 0 and w < need:
            t = blocks[b][j]
            if hit(t):
                best = w if best is None else min(best, w)
                break
            m = re.match(r"s_nop (\d+)", t)
            w += int(m.group(1)) + 1 if m else 1
            j -= 1
        else:
            if w < need:
                for p in pred[b]:
                    if seen.get(p, need) > w:
                        seen[p] = w
                        work.append((p, len(blocks[p]) - 1, w))
    return best


def lds_loads(blocks):
    return [(b, i) for b, ins in blocks.items() for i, t in enumerate(ins)
            if t.startswith("buffer_load") and t.endswith(" lds")]


def early_m0(blocks):
    """Loads into LDS less than one wait state behind a write of m0."""
    pred = predecessors(blocks)
    return [(b, blocks[b][max(0, i - 2):i + 1]) for b, i in lds_loads(blocks)
            if waits_since(blocks, pred, b, i, 1, lambda t: re.match(r"s_\w+ m0\b", t)) is not None]


def scalars(token):
    token = token.strip()
    if token == "vcc":
        return {"vcc_lo", "vcc_hi"}
    m = re.match(r"s\[(\d+):(\d+)\]$", token)
    if m:
        return {f"s{i}" for i in range(int(m.group(1)), int(m.group(2)) + 1)}
    return {token} if re.match(r"(s\d+|vcc_lo|vcc_hi|m0)$", token) else set()


def vector_written_scalars(t):
    """Scalar registers that a vector instruction writes."""
    op, _, rest = t.partition(" ")
    args = rest.split(",")
    if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
        return scalars(args[0])
    if op.startswith(("v_add_co", "v_sub_co", "v_addc_co", "v_subb_co", "v_subrev_co", "v_subbrev_co", "v_div_scale",
                      "v_mad_u64_u32", "v_mad_i64_i32")):
        return scalars(args[1])
    return set()


def early_scalars(blocks):
    """Memory accesses less than five wait states behind a vector write of one of their scalars."""
    pred, bad = predecessors(blocks), []
    for b, ins in blocks.items():
        for i, t in enumerate(ins):
            if not t.startswith(("buffer_", "global_", "flat_", "scratch_")):
                continue
            reads = set().union(*(scalars(w) for x in t.split(",") for w in x.split()))
            if reads and waits_since(blocks, pred, b, i, 5, lambda x: vector_written_scalars(x) & reads) is not None:
                bad.append((b, ins[max(0, i - 6):i + 1]))
    return bad


def vectors(token):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", token.strip())
    if m:
        return {m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    return {token.strip()} if re.match(r"[va]\d+$", token.strip()) else set()


def early_operands(blocks):
    """MFMAs less than two wait states behind a vector write (not an MFMA's) of an operand."""
    pred, bad = predecessors(blocks), []

    def written(t):
        op, _, rest = t.partition(" ")
        return vectors(rest.split(",")[0]) if op.startswith("v_") and not op.startswith("v_mfma") else set()

    for b, ins in blocks.items():
        for i, t in enumerate(ins):
            if t.startswith("v_mfma"):
                reads = set().union(*(vectors(x) for x in t.partition(" ")[2].split(",")[1:]))
                if waits_since(blocks, pred, b, i, 2, lambda x: written(x) & reads) is not None:
                    bad.append((b, ins[max(0, i - 3):i + 1]))
    return bad


LOAD = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"


def test_checker_finds_an_early_m0():
    assert early_m0({"entry": ["s_mov_b32 m0, s1", LOAD]})
    assert not early_m0({"entry": ["s_mov_b32 m0, s1", "s_nop 0", LOAD]})
    # over a branch
    assert early_m0({"entry": ["s_add_u32 m0, s1, 64"], ".LBB0_1": [LOAD, "s_cbranch_scc1 .LBB0_1"]})


def test_checker_finds_an_early_descriptor_word():
    wait = ["s_nop 0", "s_mov_b32 m0, s1", "s_nop 0"]
    assert early_scalars({"entry": ["v_readfirstlane_b32 s6, v2", *wait, LOAD]})
    assert early_scalars({"entry": ["v_readlane_b32 s4, v2, 3", *wait], ".LBB0_1": ["s_nop 0", LOAD]})
    assert not early_scalars({"entry": ["v_readfirstlane_b32 s6, v2", *wait, "s_nop 1", LOAD]})
    assert not early_scalars({"entry": ["v_readfirstlane_b32 s8, v2", LOAD]})
    assert not early_scalars({"entry": ["v_readfirstlane_b32 s9, v2", "s_mov_b32 s6, s9", "s_nop 0", LOAD]})


@pytest.mark.parametrize("source", SOURCES)
def test_m0_is_settled_before_a_load_into_lds(source):
    kernels = functions(device_asm(source))
    assert sum(len(lds_loads(b)) for b in kernels.values()) > 50
    bad = [(name[:80], x) for name, blocks in kernels.items() for x in early_m0(blocks)]
    assert not bad, (len(bad), bad[:3])


@pytest.mark.parametrize("source", SOURCES)
def test_scalars_of_memory_accesses_are_settled(source):
    kernels = functions(device_asm(source))
    bad = [(name[:80], x) for name, blocks in kernels.items() for x in early_scalars(blocks)]
    assert not bad, (len(bad), bad[:3])


def test_checker_finds_an_early_operand():
    mfma = "v_mfma_f32_16x16x32_f16 a[0:3], v[4:7], v[8:11], a[0:3]"
    assert early_operands({"entry": ["v_mov_b32_e32 v9, v2", "s_waitcnt lgkmcnt(0)", mfma]})
    assert early_operands({"entry": ["v_accvgpr_write_b32 a3, 0"], ".LBB0_1": [mfma]})
    assert not early_operands({"entry": ["v_mov_b32_e32 v9, v2", "s_nop 1", mfma, mfma]})


@pytest.mark.parametrize("source", SOURCES)
def test_operands_of_mfmas_are_settled(source):
    kernels = functions(device_asm(source))
    bad = [(name[:80], x) for name, blocks in kernels.items() for x in early_operands(blocks)]
    assert not bad, (len(bad), bad[:3])
