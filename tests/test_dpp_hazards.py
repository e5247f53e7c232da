"""Every DPP operand of the built kernels is read at least two wait states after a vector
instruction wrote it, and no EXEC write by a vector compare comes within five.  The DPP arithmetic
of the gridders is written in assembler statements, which the compiler's own hazard handling does
not look into, so another compiler could place a copy right before one."""

import os
import re
import shutil
import subprocess

import pytest

from paper_1905_03213_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READ_AFTER_WRITE = 2  # VALU writes a VGPR, a VALU DPP operand reads it
READ_AFTER_EXEC = 5   # VALU writes EXEC, any VALU DPP instruction
DPP = re.compile(r"\b(row_newbcast|row_shl|row_shr|row_ror|row_bcast|row_mirror|row_half_mirror|quad_perm|wave_)")
REGS = re.compile(r"^v(?:(\d+)|\[(\d+):(\d+)\])$")


def _vgprs(operand):
    m = REGS.match(operand.strip().strip("-|"))
    if not m:
        return range(0)
    lo = int(m.group(1) or m.group(2))
    return range(lo, int(m.group(3) or lo) + 1)


def _operands(text):
    # commas inside brackets (quad_perm:[1,0,3,2]) do not separate operands
    out, depth, cur = [], 0, ""
    for ch in text:
        depth += ch == "["
        depth -= ch == "]"
        if ch == "," and depth == 0:
            out.append(cur)
            cur = ""
        else:
            cur += ch
    out.append(cur)
    return [o.split()[0] if o.split() else "" for o in out]


def hazards(listing):
    """DPP reads too close to the write before them, over every path into a block."""
    code = []
    for line in listing.splitlines():
        line = line.split("//")[0].strip()
        m = re.match(r"^[0-9a-f]+ <(\w+)>:$", line)
        if m:
            code.append(("label", m.group(1), ""))
        elif re.match(r"^[a-z]\w+", line):
            op, _, rest = line.partition(" ")
            code.append(("op", op, rest))
    at_label, bad, n_dpp = {}, [], 0
    for last in (False, False, True):  # the states at labels settle within two passes of so short a window
        n_dpp, age, kernel = 0, {}, ""
        for kind, op, rest in code:
            if kind == "label":
                if not re.match(r"^L\d+$", op):
                    kernel, age = op, {}
                for reg, a in at_label.get((kernel, op), {}).items():
                    age[reg] = min(a, age.get(reg, a))
                continue
            ops = _operands(rest)
            if op.startswith("v_") and DPP.search(rest):
                n_dpp += 1
                near = [r for r in _vgprs(ops[1]) if age.get(r, 99) < READ_AFTER_WRITE]
                if last and (near or age.get("exec", 99) < READ_AFTER_EXEC):
                    bad.append(f"{op} {rest.strip()}")
            states = int(ops[0], 0) + 1 if op == "s_nop" else 1
            age = {r: a + states for r, a in age.items() if a + states < READ_AFTER_EXEC}
            if op.startswith("v_"):
                wrote = list(_vgprs(ops[0]))
                if "swap" in op:
                    wrote += _vgprs(ops[1])
                age.update((r, 0) for r in wrote)
                if op.startswith("v_cmpx"):
                    age["exec"] = 0
            if op.startswith(("s_branch", "s_cbranch")):
                here = at_label.setdefault((kernel, ops[0]), {})
                for r, a in age.items():
                    here[r] = min(a, here.get(r, a))
                if op == "s_branch":
                    age = {}
    return bad, n_dpp


def test_scan_sees_hazards():
    write = "v_mov_b32_e32 v3, v7\n"
    read = "v_fmac_f64_dpp v[0:1], v[2:3], v[8:9] row_newbcast:1 row_mask:0xf bank_mask:0xf// 00FF\n"
    swap = "v_permlane16_swap_b32_e32 v50, v3\n"
    other = "v_mov_b32_e32 v60, v7\n"
    assert len(hazards(write + read)[0]) == 1
    assert len(hazards(write + other + read)[0]) == 1
    assert len(hazards(swap + "s_nop 0\n" + read)[0]) == 1
    assert hazards(write + "s_nop 1\n" + read) == ([], 1)
    assert hazards(write + other + other + read) == ([], 1)
    # over a branch into the block, forwards and backwards
    assert len(hazards(write + "s_cbranch_scc1 L4\ns_nop 4\ns_nop 4\n0000 <L4>:\n" + read)[0]) == 1
    assert len(hazards("0000 <L4>:\n" + read + write + "s_branch L4\n")[0]) == 1
    assert len(hazards("v_cmpx_gt_u32_e32 v1, v40\ns_nop 2\n" + read)[0]) == 1


def test_built_kernels(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump is not installed")
    lib = build.LIB if os.path.exists(build.LIB) else build.build()
    copy = shutil.copy(lib, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(copy)], cwd=tmp_path, check=True, capture_output=True)
    total = 0
    for obj in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", f"--mcpu={build.ARCH}",
                               str(obj)], check=True, capture_output=True, text=True).stdout
        bad, n = hazards(text)
        total += n
        assert not bad, f"{obj.name}: {len(bad)} hazards, first {bad[0]}"
    assert total > 10000  # the gridders' DPP arithmetic is there
