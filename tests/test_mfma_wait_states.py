"""Wait states of the matrix instructions written as assembly (CPU): the tiled expert GEMM
is compiled to gfx950 assembly with the library's flags, and no instruction that the
compiler placed beside its asm v_mfma may touch their registers too early
(`mfma_hazards.py`).  The scan itself is checked on listings with planted mistakes."""
import os
import subprocess

import pytest

import mfma_hazards
from paper_2607_08782_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source", ["ffn.hip"])
def test_no_instruction_comes_too_close(source, tmp_path):
    out = str(tmp_path / "device.s")
    r = subprocess.run([build.HIPCC] + build.CFLAGS + ["--offload-device-only", "-S",
                                                       os.path.join(build.CSRC, source), "-o", out],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    found, seen = mfma_hazards.hazards(open(out).read())
    # three instances of the kernel, six copies of a stage's 64 products in each
    assert seen == 3 * 6 * 64
    assert not found, found[:5]


def _listing(*lines):
    out = ["kernel:"]
    for s in lines:
        out += ["\t;;#ASMSTART", "\t" + s[4:], "\t;;#ASMEND"] if s.startswith("asm ") else ["\t" + s]
    return "\n".join(out + ["\ts_endpgm", ".Lfunc_end0:"])


MFMA = "asm v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"


@pytest.mark.parametrize("lines,bad", [
    ((MFMA, "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v20, a2"), 0),
    ((MFMA, "s_nop 15", "v_accvgpr_read_b32 v20, a2"), 1),               # 17 states
    ((MFMA, "s_nop 15", "v_accvgpr_read_b32 v20, a4"), 0),               # another accumulator
    ((MFMA, "v_accvgpr_write_b32 a3, v1", "s_nop 15", "s_nop 15"), 1),   # overwritten
    ((MFMA, MFMA, "s_nop 15", "s_nop 15"), 0),                           # the next product
    ((MFMA, "asm v_mfma_f32_16x16x32_bf16 a[2:5], v[4:7], v[8:11], a[2:5]"), 1),
    (("v_mov_b32 v5, v1", "s_nop 1", MFMA), 0),
    (("v_mov_b32 v5, v1", "s_nop 0", MFMA), 1),                          # an operand just written
    (("v_mov_b32 v5, v1", "s_cbranch_scc0 .LBB0_1", "s_nop 7", ".LBB0_1:", MFMA), 1),
    ((MFMA, "s_cbranch_scc0 .LBB0_1", "s_nop 15", "s_nop 15", ".LBB0_1:",
      "v_add_f32 v1, v2, a1"), 1),                                       # by the short way round
])
def test_the_scan_finds_planted_mistakes(lines, bad):
    found, seen = mfma_hazards.hazards(_listing(*lines))
    assert seen == sum(s.startswith("asm ") for s in lines)
    assert len(found) == bad, found
