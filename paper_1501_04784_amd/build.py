"""Build ``libkbuild.so`` (the C-ABI library) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libkbuild.so")
SOURCES = [os.path.join(CSRC, f) for f in ("kb_api.hip", "kb_f64.hip", "kb_f32.hip", "kb_f32fb.hip")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # packed FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    """Compile the sources side by side, then link."""
    jobs = []
    for src in SOURCES:
        obj = os.path.splitext(src)[0] + ".o"
        cmd = [HIPCC, *FLAGS, *(extra or []), "-I", INCLUDE, "-I", CSRC, "-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        jobs.append((obj, cmd, subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.PIPE, text=True)))
    link = [HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB + ".tmp", *(obj for obj, _, _ in jobs)]
    failed = []
    for _, cmd, p in jobs:
        err = _errors(p.communicate()[1])
        if p.returncode != 0:
            failed.append(f"hipcc failed ({p.returncode}):\n{err}")
        elif verbose and err:
            print(err, file=sys.stderr)
    if not failed:
        r = subprocess.run(link, capture_output=True, text=True)
        if r.returncode != 0:
            failed.append(f"link failed ({r.returncode}):\n{r.stderr}")
    for obj, _, _ in jobs:
        if os.path.exists(obj):
            os.remove(obj)
    if failed:
        raise RuntimeError("\n".join(failed))
    os.replace(LIB + ".tmp", LIB)
    return LIB


def _errors(err: str) -> str:
    # the host pass does not know the packed-fp32 target feature; that warning is expected
    return "\n".join(l for l in err.splitlines() if "packed-fp32-ops" not in l and l.strip())


if __name__ == "__main__":
    print(build(verbose=True))
