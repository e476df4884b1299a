"""The scalar condition code around the GEMM loop's asm loads, on its gfx950 assembly.

A direct load of the 4-wave loop sets m0 with `s_add_u32`, which also writes
SCC.  The compiler must know that: otherwise it may place the statement
between an instruction that sets SCC (a loop compare, the low half of a 64-bit
address sum) and the one that reads it.  The carry of an operand address is
then lost where the sum crosses 4 GiB, or a loop's exit is missed.
"""

import re

from conftest import device_asm

READERS = ("s_cbranch_scc0", "s_cbranch_scc1", "s_cselect_b32", "s_cselect_b64", "s_addc_u32", "s_subb_u32",
           "s_cmov_b32", "s_cmov_b64")
WRITERS = re.compile(r"s_(cmp|cmpk|add|sub|addc|subb|addk|and|or|xor|andn2|orn2|nand|nor|xnor|not|abs|absdiff|lshl|"
                     r"lshr|ashr|lshl\d_add|min|max|bfe|bitcmp|bcnt|wqm|quadmask)")


def lost_conditions(lines):
    """SCC reads whose last SCC write, in program order, is the m0 addition."""
    bad, last = [], ""
    for x in lines:
        t = x.strip()
        if not t or t.startswith((";", ".", "#")):
            continue
        op = t.split()[0]
        if op in READERS and re.match(r"s_add_u32 m0\b", last):
            bad.append((last, t))
        if WRITERS.match(op):
            last = t
    return bad


def test_checker_finds_a_lost_carry():
    assert lost_conditions(["s_add_u32 s0, s0, s4", "s_add_u32 m0, s9, 1024", "s_addc_u32 s1, s1, 0"])
    assert not lost_conditions(["s_add_u32 m0, s9, 1024", "s_add_u32 s0, s0, s4", "s_addc_u32 s1, s1, 0"])


def test_no_scalar_condition_is_lost_across_a_direct_load():
    lines = device_asm("gemm_f16.hip")
    assert any("s_add_u32 m0" in x for x in lines)
    bad = lost_conditions(lines)
    assert not bad, bad[:5]
