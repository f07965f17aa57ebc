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


# the two-tile form of the 16x16x32 programs: the tiles of one key or row block, several blocks each with a mask of its own
SRC_TWO = """
#include "attn_common.h"
extern "C" __global__ void k(float* x, const int* limit) {
    sp::f32x4 t[2][2];
    for (int i = 0; i < 16; ++i) t[i / 8][i / 4 % 2][i % 4] = x[64 * i + threadIdx.x];
    for (int b = 0; b < 2; ++b) sp::hide_lanes(t[0][b], t[1][b], __builtin_amdgcn_ballot_w64(limit[64 * b + threadIdx.x] <= 7));
    for (int i = 0; i < 16; ++i) x[64 * i + threadIdx.x] = t[i / 8][i / 4 % 2][i % 4];
}
"""


@pytest.mark.parametrize("padded", [False, True])
def test_selects_on_a_mask_come_behind_its_wait(tmp_path, padded):
    check_selects(tmp_path, SRC, 1, padded)


@pytest.mark.parametrize("padded", [False, True])
def test_selects_of_two_tiles_come_behind_their_wait(tmp_path, padded):
    check_selects(tmp_path, SRC_TWO, 2, padded)


def check_selects(tmp_path, source, n_masks, padded):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    src, out = tmp_path / "k.hip", tmp_path / "k.ll"
    src.write_text(source)
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "--offload-device-only", "-std=c++17", "-S", "-emit-llvm",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "paper_2604_27089_amd", "csrc"), str(src), "-o", str(out)]
    r = subprocess.run(cmd + (["-DSP_PADDED_MFMA"] if padded else []), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = out.read_text()
    waited = set(re.findall(r"(%[\w.]+) = [^\n]*asm (?:sideeffect )?\"s_nop 1\", \"=s,0[^\n]*", text))
    selects = re.findall(r"asm (?:sideeffect )?\"([^\"]*v_cndmask_b32[^\"]*)\", \"[^\"]*\"\(([^)]*)\)", text)
    assert len(selects) == 16 and len(waited) == n_masks
    for body, args in selects:
        masks = re.findall(r"i64 (%[\w.]+)", args)
        assert masks and set(masks) <= waited, "a select may be placed before the wait for its mask"
        assert ("s_nop" in body) == padded
