"""Build libmfac.so (all HIP sources of csrc/) for gfx950 with hipcc, in place.

Usage: python -m paper_2107_03356_amd.build   (or call build()).
The shared library lands next to this file; nothing is installed elsewhere.
"""

import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmfac.so")
ARCH = os.environ.get("MFAC_OFFLOAD_ARCH", "gfx950")

SOURCES = ["pass.hip", "gram.hip", "chol.hip", "factor.hip", "static.hip", "static_query.hip", "capi.hip"]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    f"--offload-arch={ARCH}",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Compile every source to an object in _build/ and link libmfac.so."""
    out_dir = os.path.join(HERE, "_build")
    os.makedirs(out_dir, exist_ok=True)
    cc = hipcc()
    objs = []
    for src in SOURCES:
        obj = os.path.join(out_dir, src.replace(".hip", ".o"))
        cmd = [cc, *FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stderr)
            raise subprocess.CalledProcessError(r.returncode, cmd)
        # report kernels that use per-lane scratch: a staging array the
        # compiler did not keep in registers is a performance bug; the few
        # spills of the MFMA tile kernels under their 4-waves-per-SIMD launch
        # bounds (k_gram_window, k_gram_blocks, fp64 k_bgemm with a transposed
        # B) are measured wins over fewer waves without them; k_trmm32 (12 and
        # 76 bytes) keeps a few values there that it reloads once per row
        # tile, outside its k loop
        name = None
        for line in r.stderr.splitlines():
            m = re.search(r"Function Name: (\S+)", line)
            if m:
                name = m.group(1)
            m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
            if m and int(m.group(1)) > 0:
                print(f"[build] warning: {src}: {name} uses {m.group(1)} bytes/lane of scratch", file=sys.stderr)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [cc, *FLAGS, "-shared", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
