"""What the compiler cannot check for hand-written instructions, checked on the built library: a DPP operand must not
have been written by a vector instruction in the two wait states before it (the hazard recogniser does not look into
inline assembly).  Needs no GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_11305_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def violations(lines):
    """(number of DPP multiply-adds, those that read a register too early) of a disassembly."""
    recent, sites, bad = [], 0, []                       # recent: (registers written, wait states it stands for)
    for line in lines:
        line = line.split("//")[0].strip()
        if line.endswith(">:"):
            recent = []
            continue
        m = re.match(r"([a-z]\w+)\s*(.*)", line)
        if not m:
            continue
        name, operands = m.group(1), [o.strip() for o in re.sub(r"\[(\d+):(\d+)\]", r"[\1-\2]", m.group(2)).split(",")]
        if name == "v_fmac_f32_dpp":
            sites += 1
            source, age = operands[1], 0
            for written, states in reversed(recent):
                if age >= 2:
                    break
                if int(source[1:]) in written:
                    bad.append(line)
                age += states
        written = set()
        dest = re.match(r"v(\d+)$|v\[(\d+)-(\d+)\]$", operands[0]) if name.startswith("v_") else None
        if dest:
            lo, hi = (dest.group(1), dest.group(1)) if dest.group(1) else (dest.group(2), dest.group(3))
            written = set(range(int(lo), int(hi) + 1))
        recent = recent[-3:] + [(written, int(operands[0], 0) + 1 if name == "s_nop" else 1)]
    return sites, bad


def test_the_check_sees_a_violation():
    ok = ["k <f>:", "v_mov_b32_e32 v4, v1", "s_nop 1", "v_fmac_f32_dpp v53, v4, v22 row_newbcast:0 row_mask:0xf bank_mask:0xf"]
    assert violations(ok) == (1, [])
    for gap in ([], ["s_nop 0"], ["v_add_f32_e32 v9, v8, v7"]):
        assert len(violations(ok[:2] + gap + ok[3:])[1]) == 1
    assert len(violations(["v_pk_mov_b32 v[4:5], v[2:3], v[2:3]", ok[3]])[1]) == 1


def test_dpp_operands_of_the_built_library(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(B.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    code, = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    text = subprocess.run([OBJDUMP, "-d", str(tmp_path / code)], check=True, stdout=subprocess.PIPE, text=True).stdout
    sites, bad = violations(text.splitlines())
    assert sites > 1000 and not bad, bad[:5]
