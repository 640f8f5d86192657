"""csrc/grid_plan.hpp, compiled for the host: the plane sweep's plan and rule."""
import ctypes as C
import functools
import os
import subprocess
import tempfile
from dataclasses import dataclass

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2305_05988_amd", "csrc")


def build(source):
    """A shared library of C++ source, with the csrc folder to include from."""
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "t.cpp"), os.path.join(d, "t.so")
        with open(src, "w") as f:
            f.write(source)
        subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-fPIC", "-shared", "-Wall", "-I", CSRC, src,
                        "-o", lib], check=True)
        return C.CDLL(lib)


@dataclass
class Shape:
    points: int  # per thread
    W: int
    H: int
    ntx: int
    nty: int
    zb: int
    ncz: int
    fill: float

    @property
    def bricks(self):
        return self.ntx * self.nty * self.ncz


@functools.lru_cache(maxsize=None)
def _lib():
    lib = build("""
#include "grid_plan.hpp"
extern "C" double shape(int npts, int nx, int ny, int nz, int *out) {
  const its::GridShape s = its::grid_shape(npts, nx, ny, nz);
  const int v[] = {s.points, s.plan.W, s.plan.H, s.plan.ntx, s.plan.nty, s.plan.zb, s.plan.ncz};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
  return s.fill;
}
extern "C" int takes(int npts, int nx, int ny, int nz, int packed) {
  return its::grid_takes(npts, nx, ny, nz, packed != 0);
}
extern "C" int takes_cg(int npts, int nx, int ny, int nz) { return its::grid_takes_cg(npts, nx, ny, nz); }
""")
    lib.shape.restype = C.c_double
    return lib


def shape(npts, g):
    out = (C.c_int * 7)()
    fill = _lib().shape(npts, *g, out)
    return Shape(*out, fill)


def takes(npts, g, packed=False):
    return bool(_lib().takes(npts, *g, int(packed)))


def takes_cg(npts, g):
    return bool(_lib().takes_cg(npts, *g))
