"""Build libhata.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhata.so")
OBJ = os.path.join(HERE, "_build")
SOURCES = ["hata_api.hip", "hata_encode.hip", "hata_score.hip", "hata_topk.hip", "hata_attn.hip", "hata_dense.hip", "hata_gather.hip", "hata_coop.hip", "hata_unit.hip",
           "hata_train.hip", "hata_probe.hip"]
HEADERS = ["hata_device.h", "hata_internal.h", "hata_select.h", "hata_trace.h", "hata_attn_core.h", "hata_hash.h", os.path.join("..", "..", "include", "hata.h"),
           os.path.join("..", "..", "include", "hata_train.h")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]
# The first arguments of a kernel in registers when a wave starts, instead of a cold scalar load in front of its first request:
# 0.15 us a launch of the stage kernels (five calls 26.7 -> 26.0 us).  The trainer's, which wait for their rows, lose 0.5 % by it.
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]
PRELOAD_SOURCES = ["hata_encode.hip", "hata_score.hip", "hata_topk.hip"]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    return any(stale_object(s, LIB) for s in SOURCES)


def stale_object(src: str, obj: str) -> bool:
    """Older than its source, a header or this file, which holds the flags (a source's own among them)."""
    deps = [os.path.join(CSRC, s) for s in [src] + HEADERS] + [os.path.join(HERE, "build.py")]
    return not os.path.exists(obj) or any(os.path.getmtime(d) > os.path.getmtime(obj) for d in deps)


def build(force: bool = True, verbose: bool = False, trace: bool = False) -> str:
    """trace=True adds the in-kernel timestamp hooks of hata_trace.h (tuning builds only)."""
    if not force and not stale():
        return LIB
    if trace:
        cmds = [[HIPCC] + FLAGS + ["-DHATA_TRACE", "-fgpu-rdc"] + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]]
        link = None
    else:
        # one object per source, compiled side by side (objects of sources that did not change are
        # kept unless force is set), then one link
        os.makedirs(OBJ, exist_ok=True)
        compile_flags = [f for f in FLAGS if f != "-shared"] + ["-c"]
        cmds, objs = [], []
        for src in SOURCES:
            o = os.path.join(OBJ, src.replace(".hip", ".o"))
            objs.append(o)
            if force or stale_object(src, o):
                cmds.append([HIPCC] + compile_flags + (PRELOAD if src in PRELOAD_SOURCES else []) + [os.path.join(CSRC, src), "-o", o])
        link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + out)
        if verbose and out.strip():
            print(out)

    from concurrent.futures import ThreadPoolExecutor
    with ThreadPoolExecutor(max_workers=min(8, max(1, len(cmds)))) as pool:
        list(pool.map(run, cmds))
    if link:
        run(link)
    return LIB


if __name__ == "__main__":
    build(force="--changed" not in sys.argv, verbose=True, trace="--trace" in sys.argv)
    print(LIB)
