"""Inline assembly in the kernels keeps the target's wait states: a mask (VCC or
an SGPR pair) that a vector instruction writes is read by a vector instruction
only after two wait states.  The compiler sees to that in its own code, but not
between the instructions of an asm statement."""

import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1302_2669_amd", "csrc")
WAIT_STATES = 2


def asm_blocks():
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".h", ".hip", ".cpp")):
            continue
        with open(os.path.join(CSRC, name)) as fh:
            text = fh.read()
        for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
            body = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            code = [i.strip() for i in re.split(r"\\n|;", body.replace("\\t", " ")) if i.strip()]
            if code:
                yield f"{name}:{text[:m.start()].count(chr(10)) + 1}", code


def masks(instr):
    """(mask registers written, mask registers read) of one vector instruction."""
    op, _, rest = instr.partition(" ")
    args = [a.strip() for a in rest.split(",")]
    if op.startswith("v_cmp"):
        return [args[0]], []
    if op.startswith(("v_addc_co", "v_subb_co", "v_subbrev_co")):
        return [args[1]], [args[4]]
    if op.startswith(("v_add_co", "v_sub_co", "v_subrev_co")):
        return [args[1]], []
    if op.startswith("v_cndmask"):
        return [], [args[3]]
    return [], []


def violations(code):
    since, bad = {}, []
    for instr in code:
        written, read = masks(instr)
        bad += [instr for r in read if since.get(r, WAIT_STATES) < WAIT_STATES]
        m = re.match(r"s_nop\s+(\d+)", instr)
        since = {r: n + (int(m.group(1)) + 1 if m else 1) for r, n in since.items()}
        since.update({w: 0 for w in written})
    return bad


def test_violations_count_instructions_and_nops():
    cmp_, use = "v_cmp_ge_u32 vcc, %1, %2", "v_cndmask_b32 %0, 0, %3, vcc"
    assert violations([cmp_, use]) and violations([cmp_, "s_nop 0", use])
    assert not violations([cmp_, "s_nop 1", use])
    assert not violations([cmp_, "v_mov_b32 %0, 0", "v_mov_b32 %1, 0", use])
    assert violations(["v_cmp_lt_u32 %1, %2, %3", cmp_, "v_addc_co_u32 %0, %1, 0, %0, %1"])


BLOCKS = list(asm_blocks())


def test_asm_statements_are_found():
    assert len(BLOCKS) >= 4


@pytest.mark.parametrize("where,code", BLOCKS, ids=[b[0] for b in BLOCKS])
def test_masks_are_read_after_their_wait_states(where, code):
    assert violations(code) == []
