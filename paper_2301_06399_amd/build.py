"""Compile the HIP library libmpt.so for gfx950 (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OUT = os.path.join(PKG, "libmpt.so")
BUILD = os.path.join(ROOT, "_build")
ARCH = os.environ.get("MPT_OFFLOAD_ARCH", "gfx950")

FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         # no packed FP32 instructions (v_pk_*_f32) anywhere
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include")]
# One object per source, and one per (mode, form, scene in LDS) of the solver
# kernels, whose instantiations dominate the compile time.
LM = [(f"mpt_lm_{m}{f}{l}", "mpt_lm.hip", [f"-DMPT_LM_MODE={m}", f"-DMPT_LM_FORM={f}", f"-DMPT_LM_LDS={l}"])
      for m in (1, 0, 2) for f in (1, 0) for l in (1, 0)]
OBJECTS = LM + [(s, s + ".hip", []) for s in ("mpt_solve", "mpt_api", "mpt_mlp", "mpt_cand", "mpt_valid")]
# The solver fuses a multiply and an add only inside one source expression
# (fp-contract=on), never across statements: whether two operations fuse
# then depends on the source alone, not on the kernel a path function is
# inlined into, so every launch schedule runs the same per-path arithmetic.
EXTRA = {"mpt_solve.hip": ["-ffp-contract=on"], "mpt_lm.hip": ["-ffp-contract=on"]}


def _compile(unit) -> str:
    name, src, defines = unit
    obj = os.path.join(BUILD, name + ".o")
    cmd = ["hipcc", *FLAGS, *EXTRA.get(src, []), *defines, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {name}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(min(len(OBJECTS), os.cpu_count() or 1)) as ex:
        objs = list(ex.map(_compile, OBJECTS))
    tmp = OUT + ".tmp"
    cmd = ["hipcc", "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp]
    subprocess.check_call(cmd)
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
