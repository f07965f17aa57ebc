"""The order of assembly statements that the compiler may move: what a wait covers has to depend on it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
#include "attn_common.h"
extern "C" __global__ void k(float* x, const int* limit) {
    sp::f32x16 t;
    for (int r = 0; r < 16; ++r) t[r] = x[64 * r + threadIdx.x];
    sp::hide_lanes(t, __builtin_amdgcn_ballot_w64(limit[threadIdx.x] <= 7));
    for (int r = 0; r < 16; ++r) x[64 * r + threadIdx.x] = t[r];
}
"""


@pytest.mark.parametrize("padded", [False, True])
def test_selects_on_a_mask_come_behind_its_wait(tmp_path, padded):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    src, out = tmp_path / "k.hip", tmp_path / "k.ll"
    src.write_text(SRC)
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "--offload-device-only", "-std=c++17", "-S", "-emit-llvm",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "paper_2604_27089_amd", "csrc"), str(src), "-o", str(out)]
    r = subprocess.run(cmd + (["-DSP_PADDED_MFMA"] if padded else []), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = out.read_text()
    waited = set(re.findall(r"(%[\w.]+) = [^\n]*asm (?:sideeffect )?\"s_nop 1\", \"=s,0[^\n]*", text))
    selects = re.findall(r"asm (?:sideeffect )?\"([^\"]*v_cndmask_b32[^\"]*)\", \"[^\"]*\"\(([^)]*)\)", text)
    assert len(selects) == 16
    for body, args in selects:
        masks = re.findall(r"i64 (%[\w.]+)", args)
        assert masks and set(masks) <= waited, "a select may be placed before the wait for its mask"
        assert ("s_nop" in body) == padded
