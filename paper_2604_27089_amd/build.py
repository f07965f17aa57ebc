"""Build the C-ABI library: hipcc, gfx950 only, in-tree.

    python -m paper_2604_27089_amd.build

produces paper_2604_27089_amd/libsp_hotpath.so and two builds for tests next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsp_hotpath.so")
# The same sources with every hand-scheduled MFMA padded by full waits and wait states (-DSP_PADDED_MFMA):
# slow, hazard-proof, bit-identical by construction; a GPU test compares the two builds.
LIB_PADDED = os.path.join(HERE, "libsp_hotpath_padded.so")
# The same objects but for attn_bwd.hip, which sends every backward to the programs of long launches
# (-DSP_BWD_ALWAYS_LONG): GPU tests hold the edges of those programs to the oracle at small sizes.
LIB_LONG = os.path.join(HERE, "libsp_hotpath_long.so")
SOURCES = ["sp_api.hip", "relayout.hip", "doc_bounds.hip", "attn_fwd.hip", "attn_bwd.hip", "attn_bwd_d128.hip", "attn_bwd_d64.hip",
           "attn_bwd_d128_long.hip", "attn_bwd_d64_long.hip", "attn_merge.hip", "pointwise.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Wall", "-Wextra",
         "-Wno-unused-command-line-argument", "-Wno-unused-parameter",
         # keep the compiler from forming packed-fp32 VALU instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(job) -> str:
    src, suffix, defines = job
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + suffix)
    cmd = ["hipcc", *FLAGS, *defines, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "packed-fp32-ops' is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _link(objs, lib: str):
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", lib], check=True)


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    slow_first = sorted(SOURCES, key=lambda s: not s.startswith("attn_bwd_d"))
    work = [(s, ".o", []) for s in slow_first] + [(s, ".padded.o", ["-DSP_PADDED_MFMA"]) for s in slow_first]
    work.append(("attn_bwd.hip", ".long.o", ["-DSP_BWD_ALWAYS_LONG"]))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = dict(zip([(s, suffix) for s, suffix, _ in work], ex.map(_compile, work)))
    _link([objs[s, ".o"] for s in SOURCES], LIB)
    _link([objs[s, ".padded.o"] for s in SOURCES], LIB_PADDED)
    _link([objs[s, ".long.o" if s == "attn_bwd.hip" else ".o"] for s in SOURCES], LIB_LONG)
    return LIB


if __name__ == "__main__":
    print(build())
