"""Wait states that hand-written assembly has to keep, checked in the built code.

The compiler places wait states around its own instructions but does not look
inside assembly blocks, nor at what an earlier instruction left for their first
ones.  On gfx950 a register written by a vector instruction may be read through
a DPP permutation only two wait states later, and the result of a
transcendental instruction by another vector instruction one later; a read that
comes too early takes the old value without any error.

check() walks the disassembly of a library's gfx950 code along every branch.
"""
import os
import re
import struct
import subprocess
import tempfile

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
DPP_STATES, TRANS_STATES = 2, 1
TRANS = ("v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_", "v_exp_", "v_log_")
# instructions whose first operand is no vector register they write
NO_DST = ("v_cmp", "v_readlane", "v_readfirstlane", "v_nop")
_LABEL = re.compile(r"^[0-9a-f]+ <(.+)>:$")
_VREG = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")
_DPP = re.compile(r"\s(quad_perm:|row_shl:|row_shr:|row_ror:|row_newbcast:|row_bcast:|row_mirror|row_half_mirror|"
                  r"wave_shl:|wave_shr:|wave_rol:|wave_ror:)")


def code_objects(lib):
    """The gfx code objects embedded in a library."""
    data, out = open(lib, "rb").read(), []
    at = data.find(BUNDLE)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        entry = at + len(BUNDLE) + 8
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", data, entry)
            ident = data[entry + 24:entry + 24 + id_len].decode()
            entry += 24 + id_len
            if "gfx" in ident and size:
                out.append(data[at + off:at + off + size])
        at = data.find(BUNDLE, at + len(BUNDLE))
    return out


def disassemble(obj):
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "code.co")
        with open(path, "wb") as f:
            f.write(obj)
        return subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--mcpu=gfx950", "--symbolize-operands", path],
                              capture_output=True, text=True, check=True).stdout


def _regs(text):
    out = set()
    for m in _VREG.finditer(text):
        if m.group(1):
            out.add(int(m.group(1)))
        else:
            out.update(range(int(m.group(2)), int(m.group(3)) + 1))
    return frozenset(out)


def _parse(listing):
    """One tuple per line of interest: (label,) or (text, wait states, registers
    written, written by a transcendental, registers read through DPP, registers
    read, branch target, falls through)."""
    code, none = [], frozenset()
    for line in listing.splitlines():
        m = _LABEL.match(line)
        if m:
            code.append((m.group(1),))
            continue
        text = line.split("//")[0].split(";")[0].strip()
        op, _, rest = text.partition(" ")
        if not (line.startswith(("\t", " ")) and re.match(r"^[a-z]+_\w+$", op)):
            continue
        if op == "s_nop":
            code.append((text, int(rest, 0) + 1, none, False, none, none, None, True))
        elif op.startswith("s_"):
            target = rest.strip() if op == "s_branch" or op.startswith("s_cbranch") else None
            ends = op in ("s_branch", "s_endpgm", "s_setpc_b64")
            code.append((text, 1, none, False, none, none, target, not ends))
        elif not op.startswith("v_"):
            code.append((text, 1, none, False, none, none, None, True))
        else:
            m = _DPP.search(rest)
            ops = (rest[:m.start()] if m else rest).split(",")
            # (v[2:3] holds no comma, so operands split cleanly)
            dst = none if op.startswith(NO_DST) else _regs(ops[0])
            if op.startswith("v_swap"):
                dst |= _regs(ops[1])
            src = ops if op.startswith(NO_DST) or "fmac" in op or op.startswith("v_swap") else ops[1:]
            dpp = _regs(ops[1]) if m and len(ops) > 1 else none
            code.append((text, 1, dst, op.startswith(TRANS), dpp, _regs(",".join(src)), None, True))
    return code


def listing_hazards(listing):
    """(DPP instructions, [messages]) of a disassembly."""
    code = _parse(listing)
    # what is still too fresh: registers written 0 and 1 wait states ago, and those
    # by a transcendental 0 wait states ago
    fresh = (frozenset(), frozenset(), frozenset())
    into, found, dpps = {}, {}, 0
    join = lambda a, b: tuple(x | y for x, y in zip(a, b))  # noqa: E731
    changed = True
    while changed:
        changed, dpps = False, 0
        now, falls, name = fresh, False, ""
        for i, ins in enumerate(code):
            if len(ins) == 1:
                if not re.match(r"^L\d+$", ins[0]):
                    name, falls = ins[0], False
                key = (name, ins[0])
                now = join(into.get(key, fresh), now if falls else fresh)
                falls = True
                continue
            text, states, dst, trans, dpp, src, target, falls_on = ins
            if dpp:
                dpps += 1
                early = dpp & (now[0] | now[1])
                if early:
                    found[i] = f"{name}: v{min(early)} is read through DPP too early: {text}"
            if text.startswith("v_") and not trans and src & now[2]:
                found[i] = f"{name}: v{min(src & now[2])} is read right after a transcendental: {text}"
            if states >= 2:
                now = fresh
            else:
                now = (dst, now[0], dst if trans else frozenset())
            if target is not None:
                key = (name, target)
                new = join(into.get(key, fresh), now)
                if new != into.get(key):
                    into[key] = new
                    changed = True
            if not falls_on:
                now, falls = fresh, False
    return dpps, [found[i] for i in sorted(found)]


def check(lib):
    """Raise RuntimeError if the library's gfx code reads a register too early."""
    objs = code_objects(lib)
    if not objs:
        raise RuntimeError(f"{lib}: no gfx code found")
    bad = []
    for obj in objs:
        bad += listing_hazards(disassemble(obj))[1]
    if bad:
        raise RuntimeError("registers read too early:\n" + "\n".join(bad[:20]))
