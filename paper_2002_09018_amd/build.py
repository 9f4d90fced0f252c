"""Builds libshampoo.so for gfx950 with hipcc (in-tree, next to this file)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libshampoo.so")
SOURCES = [os.path.join(HERE, "csrc", "shampoo.hip")]
HEADERS = [os.path.join(HERE, "csrc", f) for f in ("kernels.hpp", "tile_mfma.hpp", "fp32_block.hpp", "split_mfma.hpp",
                                                   "direct_mma.hpp", "small_root.hpp", "embedding.hpp")]
HEADERS.append(os.path.join(ROOT, "include", "shampoo.h"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def command(out=LIB, extra=()):
    return [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
            # packed-fp32 VALU ops are kept out of the device code
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
            *extra, *SOURCES, "-o", out]


def build(verbose=False):
    tmp = LIB + ".tmp"
    cmd = command(tmp)
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building libshampoo.so")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
