"""Build in-tree: the HIP library liblx_sparse.so (gfx950) and the native part of its Python binding, _lx_call.<ABI tag>.so."""
from __future__ import annotations

import importlib.machinery
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblx_sparse.so")
# The tag of this interpreter is part of the name: another one, whose objects are laid out otherwise, finds no file.
CALL = os.path.join(HERE, "_lx_call" + importlib.machinery.EXTENSION_SUFFIXES[0])
SOURCES = ["lx_api.hip", "compact.hip", "ffn_f32.hip", "ffn_bf16.hip", "predict_bf16.hip", "lora_bf16.hip",
           "attn_bf16.hip", "attn_f32.hip", "probe.hip"]
# -Wno-inline-asm: the DMA helpers name m0 (a register the compiler reserves) as clobbered, which
# is the point, and clang warns about every such statement
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-inline-asm",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd, out) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines()
                    if "not a recognized feature" not in l)
    if r.returncode != 0:
        if os.path.exists(out):
            os.remove(out)          # never leave a stale library behind a failed build
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + err)
    if err.strip():
        sys.stderr.write(err + "\n")


def build(verbose: bool = False) -> str:
    _run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-fvisibility=hidden",
          "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "lx_call.cpp"), "-o", CALL], CALL)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, "-shared", "-Wl,--no-undefined", *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        cmd.insert(1, "-Rpass-analysis=kernel-resource-usage")
    _run(cmd, LIB)
    return LIB


def ensure() -> None:
    """Builds if any of what the package loads is not there."""
    if not (os.path.exists(LIB) and os.path.exists(CALL)):
        build()


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
