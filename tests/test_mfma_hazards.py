"""The matrix products written as inline assembly, in the machine code of the built library.

The hardware does not interlock two uses around a matrix instruction (CDNA3 instruction set manual, section 4.5): an A, B or index
register that a vector instruction wrote less than two wait states before, and a result that anything but another matrix
instruction touches before it is there (19 wait states behind the longest of these).  The compiler waits for both around its own, but
does not look into inline assembly: there it follows from where it places copies and spills, so every build is checked.
"""
import os
import re
import subprocess

import pytest

from paper_2504_02692_amd import binding as B
from paper_2504_02692_amd import build
from tests.test_dpp_hazards import OBJDUMP, parse

WAIT_OPERAND, WAIT_RESULT = 2, 19


def registers(operand):
    """VGPRs and AGPRs of an operand."""
    m = re.match(r"-?\|?([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {(m[1], r) for r in range(lo, hi + 1)}


def is_matrix(mnemonic):
    return mnemonic.startswith(("v_mfma", "v_smfmac"))


def written(mnemonic, operands):
    """Registers that a vector instruction other than a matrix one writes."""
    if not mnemonic.startswith("v_") or is_matrix(mnemonic) or mnemonic.startswith(("v_cmp", "v_readlane", "v_readfirstlane", "v_nop")) or not operands:
        return set()
    return registers(operands[0]) | (registers(operands[1]) if "swap" in mnemonic else set())


def hazards(code):
    """(number of sparse products, the instructions that come too soon)."""
    jumps = {}
    for i, (mn, ops, _) in enumerate(code):
        if mn.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(ops[-1].strip().strip("<>"), []).append(i)

    def before(i):
        out = [j for label in code[i][2] for j in jumps.get(label, [])]
        if i > 0 and code[i - 1][0] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            out.append(i - 1)
        return out

    def clash(i, touches, left):
        """Is there an instruction that `touches`, with `left` wait states still missing in front of number i?"""
        for j in before(i):
            mn, ops, _ = code[j]
            if touches(mn, ops):
                return True
            rest = left - (int(ops[0], 0) + 1 if mn == "s_nop" else 1)
            if rest > 0 and clash(j, touches, rest):
                return True
        return False

    found, sparse = [], 0
    for i, (mn, ops, _) in enumerate(code):
        if is_matrix(mn):
            sparse += mn.startswith("v_smfmac")
            used = set().union(*(registers(o) for o in ops[1:3]))
            if mn.startswith("v_smfmac"):
                used |= registers(ops[3].split()[0])
            if clash(i, lambda m, o: written(m, o) & used, WAIT_OPERAND):
                found.append(code[i])
        else:
            used = {r for o in ops for r in registers(o) if r[0] == "a"}
            if used and clash(i, lambda m, o: m.startswith("v_smfmac") and registers(o[0]) & used, WAIT_RESULT):
                found.append(code[i])
    return sparse, found


SPARSE = "v_smfmac_f32_32x32x32_bf16 a[0:15], v[2:5], v[6:13], v14"


@pytest.mark.parametrize("body,bad", [
    (SPARSE, False),
    (f"v_mov_b32_e32 v14, v20\n {SPARSE}", True),                                          # the positions
    (f"v_mov_b32_e32 v14, v20\n s_nop 1\n {SPARSE}", False),
    (f"v_mov_b32_e32 v14, v20\n s_nop 0\n {SPARSE}", True),
    (f"v_accvgpr_read_b32 v4, a99\n s_mov_b32 s0, s1\n {SPARSE}", True),                   # a fragment that had been put aside
    (f"v_mov_b32_e32 v15, v20\n {SPARSE}", False),
    (f"ds_read_b128 v[2:5], v30\n {SPARSE}", False),                                       # (loads are waited for by count)
    (f"{SPARSE}\n {SPARSE}", False),
    (f"{SPARSE}\n s_nop 15\n v_accvgpr_read_b32 v0, a3", True),
    (f"{SPARSE}\n s_nop 15\n s_nop 7\n v_accvgpr_read_b32 v0, a3", False),
    (f"{SPARSE}\n v_accvgpr_read_b32 v0, a16", False),
    (f"{SPARSE}\n v_accvgpr_mov_b32 a3, a20", True),
    (f"<L0>:\n {SPARSE}\n v_mov_b32_e32 v6, v2\n s_cbranch_scc0 <L0>", True),              # around the loop
    (f"v_mov_b32_e32 v6, v2\n s_branch <L1>\n<L0>:\n {SPARSE}\n<L1>:\n s_endpgm", False),
    ("v_mov_b32_e32 v2, v20\n v_mfma_f32_32x32x16_bf16 a[0:15], v[2:5], v[6:9], a[0:15]", True),
])
def test_the_check_itself(body, bad):
    assert bool(hazards(parse(body))[1]) == bad


def test_no_matrix_product_meets_a_register_too_soon(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        build.build(verbose=False)
    lib = tmp_path / "lib.so"
    lib.symlink_to(B.LIB_PATH)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    checked = 0
    for f in sorted(tmp_path.glob("*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(f)], check=True, capture_output=True, text=True).stdout
        n, found = hazards(parse(text))
        assert not found, (f.name, found[:4])
        checked += n
    assert checked > 200                         # (remainder_loop)
