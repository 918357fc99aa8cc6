"""Build step: compiles the HIP sources into paper_2312_11514_amd/liblif.so for gfx950."""
from __future__ import annotations

import glob
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "liblif.so")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _run(cmd, verbose):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print(" ".join(cmd), flush=True)


def build_library(verbose: bool = False) -> str:
    """Compiles every source on its own, several at a time, and links them into liblif.so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory(prefix="lif_build_") as tmp:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
        jobs = min(len(SOURCES), os.cpu_count() or 1, 8)
        with ThreadPoolExecutor(jobs) as pool:
            list(pool.map(lambda so: _run([hipcc, *HIPCC_FLAGS, "-c", "-o", so[1], so[0]], verbose), zip(SOURCES, objects)))
        linked = os.path.join(tmp, "liblif.so")
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", linked, *objects], verbose)
        with open(linked, "rb") as f, open(LIB_PATH + ".new", "wb") as g:
            g.write(f.read())
    os.chmod(LIB_PATH + ".new", 0o755)
    os.replace(LIB_PATH + ".new", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
