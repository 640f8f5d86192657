"""Build the HIP library libitsolve.so for gfx950 in-tree.

hipcc cross-compiles without a GPU.  Floating-point contraction is off, so
every fused multiply-add in the kernels is an explicit fma(); packed FP32
instructions are disabled for all device code.
"""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libitsolve.so")
SOURCES = [os.path.join(HERE, "csrc", name + ".hip") for name in ("itsolve", "batch", "grid")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False) -> str:
    """Compiles the sources side by side and links them.  The objects and the
    unfinished library have names of this call's own, so that builds at the same
    time do not write each other's."""
    tmp = f"{LIB}.tmp{os.getpid()}"
    with tempfile.TemporaryDirectory() as folder:
        objects = [os.path.join(folder, os.path.basename(src) + ".o") for src in SOURCES]
        compiles = [[HIPCC] + FLAGS + ["-c", src, "-o", obj] for src, obj in zip(SOURCES, objects)]
        link = [HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared"] + objects + ["-o", tmp]
        if verbose:
            for cmd in compiles + [link]:
                print(" ".join(cmd), flush=True)
        running = [subprocess.Popen(cmd) for cmd in compiles]
        for cmd, status in [(cmd, p.wait()) for cmd, p in zip(compiles, running)]:
            if status != 0:
                raise subprocess.CalledProcessError(status, cmd)
        subprocess.run(link, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
