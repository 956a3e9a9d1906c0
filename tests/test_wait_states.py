"""The distances that gfx950 asks for around the inline assembly of the tiled row solve, counted in the compiled code:
the compiler does not see inside assembly, so it cannot keep them there.  After a vector instruction that writes a
register: two wait states before a DPP operand or a permlane swap reads it, one before a lane read, and one between a
transcendental and another vector instruction.
"""
import os
import re
import subprocess

import pytest

from paper_2604_10377_amd import build as B

TRANS = ("v_rcp", "v_rsq", "v_sqrt", "v_exp", "v_log", "v_sin", "v_cos")


def _registers(operand):
    m = re.match(r"[-|]*v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"[-|]*v(\d+)\b", operand)
    return {int(m[1])} if m else set()


def too_close(assembly):
    """(line, instruction, distance, needed) of every read that comes too early, and the number of reads looked at."""
    bad, looked, recent = [], 0, []  # recent: [registers, transcendental, wait states since]
    for number, line in enumerate(assembly.splitlines(), 1):
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        name = text.split()[0]
        operands = [o.strip() for o in text[len(name):].split(",")]
        if name == "s_nop":
            for r in recent:
                r[2] += int(operands[0], 0) + 1
            continue
        needs = []  # (registers read, wait states needed, only after a transcendental)
        if name.startswith("v_permlane") and "swap" in name:
            needs.append((_registers(operands[0]) | _registers(operands[1]), 2, False))
        elif "_dpp" in name:
            needs.append((_registers(operands[1]), 2, False))
        elif name.startswith("v_readlane"):
            needs.append((_registers(operands[1]), 1, False))
        if name.startswith("v_") and not name.startswith(TRANS):
            needs.append((set().union(*map(_registers, operands[1:])) if len(operands) > 1 else set(), 1, True))
        for read, needed, only_trans in needs:
            looked += not only_trans
            for written, trans, age in recent:
                if written & read and age < needed and (trans or not only_trans):
                    bad.append((number, text, age, needed))
        for r in recent:
            r[2] += 1
        recent = [r for r in recent if r[2] < 2]
        if name.startswith("v_"):
            swap = name.startswith("v_permlane") and "swap" in name
            recent.append([_registers(operands[0]) | (_registers(operands[1]) if swap else set()),
                           name.startswith(TRANS), 0])
    return bad, looked


def test_too_close_sees_each_kind():
    """The counter itself, on lines with known distances."""
    for lines, bad in (("v_mov_b32_e32 v1, v2\nv_permlane16_swap_b32_e32 v1, v3", 1),
                       ("v_mov_b32_e32 v1, v2\ns_nop 0\nv_permlane16_swap_b32_e32 v3, v1", 1),
                       ("v_mov_b32_e32 v1, v2\ns_nop 1\nv_permlane16_swap_b32_e32 v1, v3", 0),
                       ("v_mul_f32_e32 v[4:5], v2, v3\nv_fmac_f32_dpp v6, v5, -v7 row_newbcast:1", 1),
                       ("v_mul_f32_e32 v5, v2, v3\nds_write_b32 v0, v1\ns_nop 0\nv_fmac_f32_dpp v6, v5, -v7 row_newbcast:1", 0),
                       ("v_fmac_f32_dpp v6, v5, -v7 row_newbcast:1\nv_readlane_b32 s0, v6, 1", 1),
                       ("v_rsq_f32_e32 v1, s0\nv_mul_f32_e32 v2, v1, v3", 1),
                       ("v_rsq_f32_e32 v1, s0\ns_nop 0\nv_mul_f32_e32 v2, v1, v3", 0)):
        assert len(too_close(lines)[0]) == bad, lines


@pytest.mark.slow
def test_tiled_row_solve(tmp_path):
    out = tmp_path / "solve_tiled.s"
    flags = [f for f in B.CFLAGS if not f.startswith("-Rpass")]
    subprocess.run([B.HIPCC] + flags + ["--cuda-device-only", "-S", os.path.join(B.CSRC, "solve_tiled.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    bad, looked = too_close(out.read_text())
    assert looked > 1000
    assert not bad, bad[:10]
