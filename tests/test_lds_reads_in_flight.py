"""The LDS reads that are written out in assembly (monarch_lds_tr.h) are waited for by the wave itself, some instructions later; the
compiler takes their registers as written at once.  So in the code it makes nothing may touch such a register, and no branch may be
passed, between the read and the next wait for all LDS accesses."""
import os
import re
import subprocess

import pytest

from paper_2204_00595_amd import build

SOURCES = ["monarch_mfma_wgrad.hip", "monarch_mfma_sq64.hip"]
_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _registers(text):
    out = set()
    for kind, lo, hi, one in _REG.findall(text):
        out |= {(kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return out


def touched_in_flight(lines):
    """(reads written out in assembly, instructions that touch one's register, or branch, before the wait)"""
    flying, written_out, reads, bad = set(), False, 0, []
    for number, line in enumerate(lines, 1):
        if "#ASMSTART" in line or "#ASMEND" in line:
            written_out = "#ASMSTART" in line
            continue
        text = line.split(";")[0].strip()
        if not text or text.endswith(":") or text.startswith("."):
            if flying and text.startswith(".LBB"):
                bad.append((number, text))
            continue
        op, _, rest = text.replace("\t", " ").partition(" ")
        if op == "s_waitcnt" and "lgkmcnt(0)" in rest:
            flying = set()
        elif flying and (_registers(rest) & flying or op.startswith(("s_cbranch", "s_branch", "s_setpc", "s_endpgm"))):
            bad.append((number, text))
        if written_out and op.startswith("ds_read"):
            reads += 1
            flying |= _registers(rest.split(",")[0])
    return reads, bad


def test_the_check_sees_what_it_looks_for():
    read = [";;#ASMSTART", "ds_read_b64_tr_b16 v[10:11], v4 offset:64", ";;#ASMEND"]
    wait = ["s_waitcnt lgkmcnt(0)"]
    assert touched_in_flight(read + ["v_mov_b32_e32 v12, v9"] + wait + ["v_mov_b32_e32 v12, v11"]) == (1, [])
    for text in ("v_mov_b32_e32 v12, v11", "v_add_u32_e32 v10, v1, v2", "v_accvgpr_write_b32 a3, v10", "s_cbranch_scc1 .LBB0_2", ".LBB0_2:"):
        assert touched_in_flight(read + [text] + wait)[1] == [(4, text)]
    assert touched_in_flight(read + ["s_waitcnt vmcnt(0)", "v_mov_b32_e32 v12, v10"])[1]
    assert touched_in_flight(["ds_read_b128 v[0:3], v9", "v_mov_b32_e32 v12, v1"]) == (0, [])   # the compiler's own: it waits


@pytest.mark.parametrize("source", SOURCES)
def test_no_register_of_a_read_in_flight_is_touched(source, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "device.s"
    subprocess.check_call([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, source)],
                          stderr=subprocess.DEVNULL)
    reads, bad = touched_in_flight(out.read_text().splitlines())
    assert reads > 0 and not bad, (reads, bad[:5])
