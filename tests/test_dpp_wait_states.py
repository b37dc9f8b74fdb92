"""Data-parallel operands (DPP) in the compiled Cholesky kernels: a vector register may be read through one only with two other
instructions or wait states behind the vector instruction that wrote it, and the result of a reciprocal or square root
only with one by any other vector instruction.  The hardware does not check either, and the compiler does not look into
hand-written statements.  So a statement has to keep to both whatever stands in front of it: here every register counts as
written right before it begins."""
import os
import re
import subprocess

import pytest

from paper_2504_05295_amd import build

DPP = re.compile(r"\b(row_newbcast|row_bcast|row_shl|row_shr|row_ror|row_share|row_xmask|quad_perm|wave_\w+|row_mirror|row_half_mirror)\b")
TRANS = re.compile(r"^v_(rcp|rsq|sqrt|exp|log|sin|cos)_")


def registers(operand):
    m = re.match(r"^\s*[-|]*v(\d+)\b", operand)
    if m:
        return {int(m.group(1))}
    m = re.match(r"^\s*[-|]*v\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


def faults(text):
    """(number of DPP reads, number of those in hand-written statements, what comes too early)"""
    found, dpp, by_hand, inside = [], 0, 0, False
    written = []        # newest last: (registers, a reciprocal or the like, wait states it stands for); None: all registers
    for number, line in enumerate(text.splitlines(), 1):
        if ";#ASMSTART" in line:
            inside = True
            written = [(None, True, 1)]
            continue
        if ";#ASMEND" in line:
            inside = False
            written = [w for w in written if w[0] is not None]    # (in front of what follows stands what was really written)
            continue
        line = line.split(";")[0].strip()
        if not line or line.startswith((".", "#", "//")) or line.endswith(":"):
            if line.endswith(":"):
                written = []    # (a join: the compiler's own instructions look after themselves)
            continue
        op, _, rest = line.partition(" ")
        operands = rest.split(",")
        is_dpp = bool(DPP.search(rest))
        dpp += is_dpp
        by_hand += is_dpp and inside
        if op.startswith("v_"):
            tied = op.startswith(("v_fmac", "v_mfma"))
            sources = [registers(o) for o in (operands if tied else operands[1:])]
            between = 0
            for regs, trans, states in reversed(written):
                if between >= 2:
                    break
                # (the first source is the one that is read through DPP)
                if is_dpp and (regs is None or regs & registers(operands[1])):
                    found.append((number, line, "data-parallel operand", between))
                if trans and between < 1 and not TRANS.match(op) and any(s if regs is None else regs & s for s in sources):
                    found.append((number, line, "result of a reciprocal", between))
                between += states
        if op == "s_nop":
            written.append((set(), False, int(operands[0]) + 1))
        else:
            out = registers(operands[0]) if op.startswith("v_") else set()
            if "swap" in op:
                out |= registers(operands[1])
            written.append((out, bool(TRANS.match(op)), 1))
        written = written[-4:]
    return dpp, by_hand, found


FMAC = "v_fmac_f32_dpp v1, v2, v3 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"


@pytest.mark.parametrize("text,count", [
    ("v_mov_b32_e32 v2, v9\n" + FMAC, 1),
    ("v_mov_b32_e32 v2, v9\nv_mov_b32_e32 v8, v9\n" + FMAC, 1),
    ("v_mov_b32_e32 v2, v9\ns_nop 1\n" + FMAC, 0),
    ("v_mov_b32_e32 v3, v9\n" + FMAC, 0),
    (";#ASMSTART\nv_add_f32 v8, v8, v8\n" + FMAC + ";#ASMEND\n", 2),
    (";#ASMSTART\ns_nop 0\nv_add_f32 v8, v8, v8\n" + FMAC + ";#ASMEND\n", 0),
    (";#ASMSTART\ns_nop 1\n" + FMAC + FMAC.replace("v2, v3", "v1, v3") + ";#ASMEND\n", 1),
    ("v_rcp_f32 v8, v9\nv_mul_f32 v7, v8, v8\n", 1),
    ("v_rcp_f32 v8, v9\ns_nop 0\nv_mul_f32 v7, v8, v8\n", 0),
])
def test_the_check(text, count):
    assert len(faults(text)[2]) == count


def test_cholesky_kernels(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "chol_panel.s")
    subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "chol_panel.hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    dpp, by_hand, found = faults(open(out).read())
    assert by_hand > 1000 and dpp > by_hand
    assert not found, (len(found), found[:5])
