"""Wait states of the built kernels' instructions (CPU only).

The kernels' instruction blocks (inline assembly) are opaque to the compiler, which inserts no
wait states inside them or between them and what follows.  This test reads the
disassembly of the built library's own code objects and holds every straight run of instructions
to the rules that the compiler applies to its own code for gfx950, in wait states between the
two instructions (an instruction is one, s_nop N is N + 1):
  - a vector register written by the VALU and read through a DPP control: 2;
  - an SGPR or VCC written by the VALU and read by the VALU (carry, select mask, constant): 2;
  - the result of a transcendental instruction and a VALU read of it: 1.
A run ends at a branch that is always taken; entries from elsewhere are not followed.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_27351_amd", "libwf.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

REG = re.compile(r"\b([sv])(\d+)\b|\b([sv])\[(\d+):(\d+)\]|\b(vcc)\b")
TRANS = re.compile(r"v_(exp|log|rcp|rsq|sqrt|sin|cos)_")
# instructions with a second destination: carry or scale out
TWO_DST = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64_")


def regs(text):
    out = set()
    for m in REG.finditer(text):
        if m.group(6):
            out.add("vcc")
        elif m.group(1):
            out.add(m.group(1) + m.group(2))
        else:
            out.update(f"{m.group(3)}{k}" for k in range(int(m.group(4)), int(m.group(5)) + 1))
    return out


def violations(lines):
    """(line, rule, register, wait states) of every pair in 'lines' (disassembly) that is too close."""
    found = []
    recent = []  # (age in wait states, VALU destinations, transcendental)
    for line in lines:
        text = line.split("//")[0].strip()
        if not text or text.endswith(":") or not re.match(r"[a-z]", text):
            continue
        op, _, rest = text.partition(" ")
        if op == "s_nop":
            recent = [(a + int(rest, 0) + 1, d, t) for a, d, t in recent]
            continue
        dst = set()
        if op.startswith("v_"):
            ops = rest.split(",")
            nd = 2 if TWO_DST.match(op) else 1
            dst, src = regs(",".join(ops[:nd])), regs(",".join(ops[nd:]))
            first = regs(ops[1]) if "_dpp" in op else set()
            if "_dpp" in op and nd == 2:
                first = regs(ops[2])
            for age, d, t in recent:
                for r in d:
                    if age < 2 and r in first and r[0] == "v" and r != "vcc":
                        found.append((text, "dpp", r, age))
                    if age < 2 and r in src and (r[0] == "s" or r == "vcc"):
                        found.append((text, "sgpr", r, age))
                    if age < 1 and t and r in src:
                        found.append((text, "trans", r, age))
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            recent = []
            continue
        recent = [(a + 1, d, t) for a, d, t in recent if a < 2]
        # what this instruction overwrites is no longer the earlier one's
        recent = [(a, d - dst, t) for a, d, t in recent]
        if dst:
            recent.append((0, dst, bool(TRANS.match(op))))
    return found


def disassembly(tmp):
    """Disassembly lines of the library's gfx950 code objects."""
    lib = os.path.join(tmp, "lib.so")
    shutil.copyfile(LIB, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=tmp)
    objs = sorted(f for f in os.listdir(tmp) if f.startswith("lib.so.") and "gfx950" in f)
    assert objs
    for f in objs:
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(tmp, f)], check=True,
                             stdout=subprocess.PIPE, text=True).stdout
        yield f, out.splitlines()


def test_the_reader_sees_each_rule():
    assert [v[1] for v in violations(["v_add_f32_e32 v1, v2, v3", "s_nop 0",
                                      "v_mov_b32_dpp v4, v1 wave_shr:1 row_mask:0xf bank_mask:0xf"])] == ["dpp"]
    assert [v[1] for v in violations(["v_cmp_lt_f32_e32 vcc, v1, v2",
                                      "v_addc_co_u32_e32 v3, vcc, v3, v3, vcc"])] == ["sgpr"]
    assert {v[1] for v in violations(["v_cmp_lt_f32_e64 s[4:5], v1, v2", "v_add_f32_e32 v1, v2, v3",
                                      "v_cndmask_b32_e64 v3, v4, v5, s[4:5]"])} == {"sgpr"}
    assert [v[1] for v in violations(["v_exp_f32_e32 v1, v2", "v_add_f32_e32 v3, 1.0, v1"])] == ["trans"]
    assert violations(["v_add_f32_e32 v1, v2, v3", "s_nop 1",
                       "v_mov_b32_dpp v4, v1 wave_shr:1 row_mask:0xf bank_mask:0xf",
                       "v_cmp_lt_f32_e32 vcc, v1, v2", "v_exp_f32_e32 v7, v2", "v_mov_b32_e32 v5, v1",
                       "v_addc_co_u32_e32 v3, vcc, v3, v3, vcc", "v_add_f32_e32 v3, 1.0, v7"]) == []


def test_built_kernels_keep_the_wait_states(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not found")
    assert os.path.exists(LIB), "build the library first"
    for name, lines in disassembly(str(tmp_path)):
        bad = violations(lines)
        assert not bad, (name, len(bad), bad[:5])
