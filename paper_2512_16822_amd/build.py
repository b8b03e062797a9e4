"""Build step: compile the HIP/C++ sources under csrc/ into libmepic.so for gfx950, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmepic.so")
SOURCES = ["pool.cpp", "attn_api.hip", "attn_combine.hip", "attn_decode_f32.hip", "attn_prefill_split.hip", "attn_decode_split.hip", "attn_decode_plain.hip", "attn_decode_batched.hip", "attn_prefill_mfma.hip", "kv_commit.hip", "decode_plan.cpp", "probes.hip"]
# -packed-fp32-ops off: hipcc must not form v_pk_*_f32 from float code on these machines.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False, jobs: int = 8, extra_flags=(), out: str = LIB, objdir: str = "") -> str:
    """Compile every source (always) and link the shared library (default: libmepic.so beside this file).
    `extra_flags` (e.g. -D tuning constants) and `out` exist for experiments; the product build uses neither."""
    objdir = objdir or os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs, objs = [], []
    for src in SOURCES:
        obj = os.path.join(objdir, src + ".o")
        objs.append(obj)
        cmd = [hipcc(), *FLAGS, *extra_flags, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    subprocess.check_call([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out, *objs])
    return out


def _drain(procs) -> None:
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        # hipcc's host pass does not know the packed-fp32 target feature and says so: harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if out:
            print(f"[{src}]\n{out}", file=sys.stderr)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
