"""Waits that the hardware does not make by itself, in the assembly of the block LDL: an instruction that reads a vector
register across lanes (DPP) stands at least two wait states behind the vector instruction that wrote it.  The compiler
sees to that for its own instructions only, and the pivots are written as text.  (A vector or scalar instruction is a wait state,
s_nop N is N + 1; straight through labels, which can only bring a write nearer than it is.)"""
import os
import re
import subprocess

import pytest

from paper_2406_11235_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ACROSS = re.compile(r"row_newbcast|row_bcast|row_sh[lr]|row_ror|row_share|row_(half_)?mirror|quad_perm|wave_")


def registers(operand):
    out = set()
    for one, first, last in re.findall(r"\bv(?:(\d+)|\[(\d+):(\d+)\])", operand):
        out |= {int(one)} if one else set(range(int(first), int(last) + 1))
    return out


def too_early(lines):
    """(reads across lanes, those less than two wait states behind the write of what they read)"""
    reads, found = 0, []
    behind = []  # (wait states, registers written by the vector ALU, text)
    for line in lines:
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        name, _, rest = text.partition(" ")
        operands = re.split(r",(?![^\[]*\])", rest)
        if name.startswith("v_") and ACROSS.search(rest):
            reads += 1
            states = 0
            for waits, written, before in reversed(behind):
                if states >= 2:
                    break
                if written & registers(operands[1].split()[0]):
                    found.append((before, text))
                states += waits
        written = set()
        if name.startswith("v_") and not name.startswith(("v_cmp", "v_readlane", "v_readfirstlane")):
            written = registers(operands[0]) | (registers(operands[1]) if "swap" in name else set())
        behind = behind[-3:] + [(int(operands[0], 0) + 1 if name == "s_nop" else 1, written, text)]
    return reads, found


def test_the_check_itself():
    swap, read = "v_permlane32_swap_b32_e32 v71, v59", "v_fmac_f64_dpp v[70:71], v[70:71], v[0:1] row_newbcast:0 row_mask:0xf"
    for between, count in (([], 1), (["v_add_f32_e32 v9, v8, v7"], 1), (["s_nop 0"], 1), (["s_nop 1"], 0),
                           ([".LBB0_1:", "s_mov_b32 s0, 1 ; c", "v_mov_b32_e32 v3, v2"], 0)):
        assert [len(f) if i else f for i, f in enumerate(too_early([swap] + between + [read]))] == [1, count]


def test_reads_across_lanes_in_the_block_ldl(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "ldlq.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-pthread")]
    subprocess.run([HIPCC] + flags + ["-S", "--cuda-device-only", "-x", "hip", os.path.join(build.CSRC, "qtip_ldlq.hip"),
                                      "-o", str(out)], check=True, capture_output=True)
    reads, found = too_early(out.read_text().splitlines())
    assert reads >= 15 * 16  # the columns of a block's pivots
    assert not found, found[:4]
