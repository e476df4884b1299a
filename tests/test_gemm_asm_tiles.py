"""Register-safety checks of every tile size of the 4-wave GEMM loop, on its gfx950 assembly.

The rules are those of the 256x256 form: nothing but an MFMA touches a
register whose LDS read has not been waited for, and nothing but an MFMA
touches an accumulator between the last MFMA and the wait states.  The
smaller tiles hold 3 to 8 LDS stages and compute their fragment addresses
inside the loop, so address arithmetic must keep out of these windows too.
"""

import re

import pytest

import test_gemm_asm_order as order
from conftest import device_asm

TILES = [(256, 256, 2), (256, 128, 3), (128, 256, 3), (128, 128, 4), (64, 64, 8)]


@pytest.fixture(scope="module")
def all_kernels():
    lines = device_asm("gemm_f16.hip")
    found = {}
    for i, line in enumerate(lines):
        if line.startswith("_Z") and "gemm_f16_kernelI" in line and line.split()[0].endswith(":"):
            end = next(j for j in range(i, len(lines)) if lines[j].startswith(".Lfunc_end"))
            found[line.split(":")[0]] = lines[i + 1:end]
    return found


def _of_tile(kernels, bm, bn, ns):
    tag = f"gemm_f16_kernelILi{bm}ELi{bn}ELi2ELi2ELi64ELi{ns}E"
    # (the ragged-K instantiations, RK = true, are compiler-scheduled)
    return {n: b for n, b in kernels.items() if tag in n and not re.search(r"ELi\dELb1EE", n)}


@pytest.mark.parametrize("bm,bn,ns", TILES)
def test_tile_is_safe(all_kernels, bm, bn, ns):
    ks = _of_tile(all_kernels, bm, bn, ns)
    tags = ["Lb0ELb1ELi0E", "Lb0ELb0ELi0E", "Lb1ELb0ELi0E", "Lb1ELb1ELi0E", "Lb0ELb1ELi1E", "Lb0ELb0ELi2E"]
    assert not [t for t in tags if t not in " ".join(ks)]
    order.test_no_accumulator_read_between_an_mfma_and_the_wait_states(ks)
    bad = []
    nm = 2 * (bm // 32) * (bn // 32)        # MFMAs of a slice
    for name, body in ks.items():
        ins = order._instructions(body)
        loops = [b for b in order._blocks(body).values() if sum(t.startswith("v_mfma") for t in b) >= nm]
        assert loops, name
        for b in loops:     # partial waits count LDS reads only: no scalar load may share the counter
            bad += [(name[-60:], t) for t in b if t.startswith(("s_load", "s_buffer_load", "ds_write"))]
        for seq in [ins] + [b + b for b in loops]:
            pending = []            # destination registers of the reads in flight, oldest first
            for t in seq:
                op = t.split()[0]
                toks = [x.rstrip(",") for x in t.split()[1:]]
                m = re.search(r"lgkmcnt\((\d+)\)", t)
                if op == "s_waitcnt" and m:
                    n = int(m.group(1))
                    pending = pending[len(pending) - n:] if 0 < n < len(pending) else pending if n else []
                    continue
                # neither operands (of MFMAs: fragments must have landed) nor
                # results nor addresses may be registers of a read in flight
                if not op.startswith("s_"):
                    busy = set().union(*pending) if pending else set()
                    if any(order._regs(x) & busy for x in toks):
                        bad.append((name[-60:], t))
                if op.startswith("ds_read"):
                    pending.append(order._regs(toks[0]))
    assert not bad, bad[:5]
