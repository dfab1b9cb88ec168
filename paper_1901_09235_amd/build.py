"""Builds the gfx950 HIP library in-tree: paper_1901_09235_amd/_build/libdicodile_mi355x.so.

    python -m paper_1901_09235_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_build")
LIB_NAME = "libdicodile_mi355x.so"
LIB_PATH = os.path.join(OUT_DIR, LIB_NAME)
# (source, definitions, object): compiled side by side, then linked
SOURCES = [("capi.hip", [], "capi.o")] + [
    ("rounds.hip", [f"-DDCDL_R={r}", f"-DDCDL_NT={nt}"], f"rounds_{r}_{nt}.o")
    for r in ("float", "double") for nt in (256, 1024)]
HEADERS = ["dcdl_device.h", "dcdl_kernels.h", "dcdl_mfma.h", "dcdl_check.h", "dcdl_fft.h", "mfma_host.inc", "batch.inc",
           "tune.inc", "dict.inc", "serve.inc", "dcdl_dict.h"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    "-munsafe-fp-atomics",
    # packed FP32 instructions stay disabled on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False) -> str:
    """Compile every HIP source into the shared library (always recompiles)."""
    os.makedirs(OUT_DIR, exist_ok=True)
    tmp = LIB_PATH + ".tmp"
    cmds = [[HIPCC] + FLAGS + defs + ["-I", os.path.join(ROOT, "include"), "-c", "-o", os.path.join(OUT_DIR, obj),
                                      os.path.join(CSRC, src)] for src, defs, obj in SOURCES]
    link = [HIPCC] + FLAGS + ["-shared", "-o", tmp] + [os.path.join(OUT_DIR, obj) for _, _, obj in SOURCES]
    runs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        runs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    outs = [(r.communicate()[0], r.returncode) for r in runs]
    if all(rc == 0 for _, rc in outs):
        if verbose:
            print(" ".join(link), flush=True)
        res = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        outs = [(res.stdout, res.returncode)]
    for out, rc in outs:
        if rc != 0:
            sys.stderr.write(out)
            raise RuntimeError(f"hipcc failed with exit code {rc}")
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
