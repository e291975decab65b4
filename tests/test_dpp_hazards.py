"""The broadcasts written as inline assembly, in the machine code of the built library.

A DPP operand read less than two wait states after a VALU instruction wrote its register is a hazard that the hardware does not
interlock (CDNA3 instruction set manual, section 4.5).  The compiler puts waits in front of the DPP instructions that it makes
itself, but does not look into inline assembly: there the distance follows from where it places copies and the instructions
around them, with this compiler and these flags.  So every build is checked.
"""
import os
import re
import subprocess

import pytest

from paper_2504_02692_amd import binding as B
from paper_2504_02692_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 2


def registers(operand):
    m = re.match(r"-?\|?v(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def parse(text):
    """(mnemonic, operands, labels in front of it) of every instruction, in order."""
    out, labels = [], []
    for line in text.splitlines():
        line = line.split("//")[0].strip()
        m = re.match(r"(?:[0-9a-f]+ )?<(\S+)>:$", line)
        if m:
            labels.append(m[1])
            continue
        m = re.match(r"([a-z]\w*)\s*(.*)$", line)
        if m and not line.endswith(":"):
            out.append((m[1], [o for o in m[2].split(",")] if m[2] else [], labels))
            labels = []
    return out


def written(mnemonic, operands):
    """VGPRs that a VALU instruction writes."""
    if not mnemonic.startswith("v_") or mnemonic.startswith(("v_cmp", "v_readlane", "v_readfirstlane", "v_nop")) or not operands:
        return set()
    return registers(operands[0]) | (registers(operands[1]) if "swap" in mnemonic else set())


def hazards(code):
    """(number of DPP instructions, those whose DPP operand is written too shortly before)."""
    jumps = {}
    for i, (mn, ops, _) in enumerate(code):
        if mn.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(ops[-1].strip().strip("<>"), []).append(i)

    def clash(i, regs, left):
        """Does an instruction that may run just before number i, with `left` wait states still missing, write one of regs?"""
        before = [j for label in code[i][2] for j in jumps.get(label, [])]
        if i > 0 and code[i - 1][0] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before.append(i - 1)
        for j in before:
            mn, ops, _ = code[j]
            if written(mn, ops) & regs:
                return True
            rest = left - (int(ops[0], 0) + 1 if mn == "s_nop" else 1)
            if rest > 0 and clash(j, regs, rest):
                return True
        return False

    found = [i for i, (mn, ops, _) in enumerate(code) if mn.endswith("_dpp")]
    return len(found), [code[i] for i in found if clash(i, registers(code[i][1][1]), WAIT_STATES)]


@pytest.mark.parametrize("body,bad", [
    ("v_mov_b32_e32 v1, v2\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", True),
    ("v_mov_b32_e32 v1, v2\n s_mov_b32 s0, s1\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", True),
    ("v_mov_b32_e32 v1, v2\n s_mov_b32 s0, s1\n v_add_f32_e32 v5, v6, v7\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", False),
    ("v_mov_b32_e32 v1, v2\n s_nop 1\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", False),
    ("v_mov_b32_e32 v4, v2\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", False),            # not the DPP operand
    ("v_mul_f64 v[2:3], v[4:5], v[6:7]\n v_fmac_f64_dpp v[8:9], -v[2:3], v[4:5] row_newbcast:1", True),
    ("v_permlane32_swap_b32_e32 v9, v1\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", True),
    ("v_cmp_gt_f32_e32 vcc, v1, v2\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0", False),
    ("<L0>:\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0\n v_mov_b32_e32 v1, v2\n s_cbranch_scc0 <L0>", True),   # around the loop
    ("v_mov_b32_e32 v1, v2\n s_branch <L1>\n<L0>:\n v_fmac_f32_dpp v3, v1, v4 row_newbcast:0\n<L1>:\n s_endpgm", False),
])
def test_the_check_itself(body, bad):
    n, found = hazards(parse(body))
    assert n == 1 and bool(found) == bad


def test_no_dpp_operand_is_written_just_before_its_use(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        build.build(verbose=False)
    lib = tmp_path / "lib.so"
    lib.symlink_to(B.LIB_PATH)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    checked = 0
    for f in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(f)], check=True, capture_output=True,
                              text=True).stdout
        n, found = hazards(parse(text))
        assert not found, (f.name, found[:4])
        checked += n
    assert checked > 1000                        # (the column steps and the 16 x 16 factorisation)
