"""Build libpagedattn.so in-tree with hipcc for gfx950 (cross-compiles without a GPU).

    python -m paper_2506_07311_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpagedattn.so")
SOURCES = ["api.hip", "kv_copy.hip", "attention_generic.hip", "attention_f32.hip", "merge.hip", "decode_mfma.hip", "decode_mfma_d64.hip",
           "decode_mfma_d256.hip", "prefill_mfma.hip", "prefill_mfma_d64.hip", "prefill_mfma_d256.hip",
           "prefill_mfma_odd.hip", "jagged_mfma.hip", "page_pool.hip"]
HEADERS = [os.path.join(CSRC, "common.h"), os.path.join(CSRC, "prefill_tiles.h"),
           os.path.join(CSRC, "decode_mfma_impl.h"), os.path.join(CSRC, "prefill_mfma_impl.h"),
           os.path.join(HERE, "..", "include", "pagedattn.h"), os.path.join(HERE, "..", "include", "pagedattn_mods.h")]
# packed-fp32 VALU forms are disabled on purpose (they have produced wrong results on these machines)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option"]


def _hipcc() -> str:
    for p in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if p and (os.path.isabs(p) and os.path.exists(p) or not os.path.isabs(p)):
            return p
    return "hipcc"


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    path = os.path.join(CSRC, src)
    deps = [path] + HEADERS
    if not force and os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(p) for p in deps):
        return obj
    cmd = [_hipcc(), *FLAGS, "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    warn = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    if warn:
        sys.stderr.write("\n".join(warn) + "\n")
    return obj


def build(force: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
    if force or not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(o) for o in objs):
        cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
        subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
