"""Wait states of the hand-written assembly: the checker itself, the rule every
block keeps towards what the compiler may place before it, and the built code."""
import os
import re

import pytest

from paper_2511_19204_amd import build, hazards

CSRC = os.path.join(os.path.dirname(build.__file__), "csrc")


def _listing(*lines):
    return "\n".join(["0000000000001900 <kernel>:"] + [ln if ln.endswith(":") else "\t" + ln for ln in lines]) + "\n"


@pytest.mark.parametrize("bad,lines", [
    (True, ["v_mov_b32_e32 v1, v2", "v_mul_f32_dpp v3, v1, v4 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf"]),
    (True, ["v_mov_b32_e32 v1, v2", "s_nop 0", "v_mov_b32_dpp v3, -v1 row_shl:4 row_mask:0xf bank_mask:0xf"]),
    (True, ["v_fma_f32 v[4:5], v2, v2, v2", "v_add_f32_e32 v9, v9, v9", "v_fmac_f32_dpp v3, v5, v4 row_newbcast:1"]),
    (True, ["v_accvgpr_read_b32 v1, a7", "v_mov_b32_dpp v3, v1 quad_perm:[1,2,0,0] row_mask:0xf bank_mask:0xf"]),
    (True, ["v_rcp_f32_e32 v1, v2", "v_mul_f32_e32 v3, v4, v1"]),
    (True, ["v_mov_b32_e32 v1, v2", "s_cbranch_scc0 L0", "s_nop 1", "0000000000001908 <L0>:",
            "v_mov_b32_dpp v3, v1 quad_perm:[0,0,0,0]"]),
    (True, ["s_nop 1", "0000000000001908 <L0>:", "v_mov_b32_dpp v3, v1 quad_perm:[0,0,0,0]", "v_mov_b32_e32 v1, v3",
            "s_cbranch_scc0 L0"]),
    (False, ["v_mov_b32_e32 v1, v2", "s_nop 1", "v_mov_b32_dpp v3, v1 quad_perm:[0,0,0,0]"]),
    (False, ["v_mov_b32_e32 v1, v2", "s_mov_b32 s0, 0", "ds_read_b32 v9, v8",
             "v_mov_b32_dpp v3, v1 quad_perm:[0,0,0,0]"]),
    # only the first source goes through the permutation; the destination of a mul is not read
    (False, ["v_mov_b32_e32 v4, v2", "v_mul_f32_dpp v4, v1, v4 quad_perm:[0,0,0,0]"]),
    (False, ["v_rcp_f32_e32 v1, v2", "v_rsq_f32_e32 v3, v1", "s_nop 0", "v_add_f32_e32 v5, v3, v1"]),
    (False, ["v_mov_b32_e32 v1, v2", "s_branch L1", "0000000000001908 <L0>:", "v_mov_b32_dpp v3, v1 quad_perm:[0,0,0,0]",
             "0000000000001910 <L1>:", "s_endpgm"]),
])
def test_checker(bad, lines):
    assert bool(hazards.listing_hazards(_listing(*lines))[1]) == bad


def _asm_blocks(path):
    """(line, instructions, operands read or written) of the assembly blocks of a
    source file, its string macros expanded."""
    text = open(path).read()
    macros = dict(re.findall(r'^#define (\w+) ("(?:[^"\\]|\\.)*")\s*$', text, re.M))
    out = []
    for m in re.finditer(r"\basm(?: volatile)?\(", text):
        code, at = "", m.end()
        while True:
            tok = re.compile(r'\s+|//[^\n]*|"((?:[^"\\]|\\.)*)"|(\w+)|([:)])').match(text, at)
            at = tok.end()
            if tok.group(3):
                break
            if tok.group(2):
                code += macros[tok.group(2)][1:-1]
            elif tok.group(1) is not None:
                code += tok.group(1)
        code = re.sub(r"%(\d+)", r"v\1", code.replace("\\n", "\n"))
        out.append((text.count("\n", 0, m.start()) + 1, [ln.strip() for ln in code.split("\n") if ln.strip()]))
    return out


def test_blocks_wait_for_what_precedes_them():
    """The instruction before a block may have written any of its operands (a copy of
    the register allocator's, a value of the compiler's): no block reads one through
    DPP in its first two wait states, nor its own results too early."""
    dpp = 0
    for name in sorted(os.listdir(CSRC)):
        for line, code in _asm_blocks(os.path.join(CSRC, name)):
            regs = sorted({int(r) for c in code for r in re.findall(r"\bv(\d+)\b", c)})
            for r in [None] + regs:
                before = [] if r is None else [f"v_mov_b32_e32 v{r}, v999"]
                n, bad = hazards.listing_hazards(_listing(*before, *code))
                assert not bad, f"{name}:{line}, operand {r}: {bad}"
            dpp += n
    assert dpp > 200  # (the path kernel's blocks were found)


def test_built_code_keeps_its_wait_states():
    assert os.path.exists(build.LIB), "build the library first"
    objs = hazards.code_objects(build.LIB)
    assert len(objs) == len(build.SOURCES)
    hazards.check(build.LIB)
