"""The iterations launched between two reads of the State (csrc/poll.hpp,
compiled for the host)."""
import ctypes as C
import math

import pytest

from . import grid_plan

MILLION = 1 << 20


@pytest.fixture(scope="module")
def lib():
    lib = grid_plan.build("""
#include "poll.hpp"
extern "C" void batches(int check_every, long n, int *out) {
  const its::Batches b = its::batches(check_every, n);
  out[0] = b.least;
  out[1] = b.most;
}
extern "C" int next_batch(int least, int most, double rho0, double rho1, long done, double thr2) {
  return its::next_batch(its::Batches{least, most}, rho0, rho1, done, thr2);
}
""")
    lib.next_batch.argtypes = [C.c_int, C.c_int, C.c_double, C.c_double, C.c_long, C.c_double]
    return lib


def _batches(lib, check_every, n):
    out = (C.c_int * 2)()
    lib.batches(check_every, C.c_long(n), out)
    return tuple(out)


def test_first_batch(lib):
    assert _batches(lib, 0, MILLION) == (8, 32)
    assert _batches(lib, 0, MILLION - 1) == (32, 32)
    assert _batches(lib, 5, MILLION) == (5, 5)


@pytest.mark.parametrize("rate", [0.01, 0.1, 0.5])
@pytest.mark.parametrize("stop", [1, 7, 8, 9, 20, 40, 100, 1000])
def test_launched_in_vain(lib, rate, stop):
    """At a steady rate no more than 8 iterations are launched in vain, and a
    long solve reads the State seldom."""
    thr2 = math.exp(-rate * stop)
    b, at, reads = 8, 0, 0
    while at < stop:
        at += b
        reads += 1
        b = lib.next_batch(8, 32, 1.0, math.exp(-rate * at), at, thr2)
        assert 8 <= b <= 32
    assert at - stop <= 8
    assert reads <= 2 + stop / 32 + 3


def test_values_that_say_nothing(lib):
    inf, nan = math.inf, math.nan
    for rho0, rho1, done in ((1.0, nan, 8), (1.0, inf, 8), (0.0, 1.0, 8), (nan, 0.5, 8), (1.0, 0.5, 0), (1.0, 1e-9, 8)):
        assert lib.next_batch(8, 32, rho0, rho1, done, 1e-8) == 8
    assert lib.next_batch(8, 32, 1.0, 0.5, 8, 0.0) == 32  # no threshold
    assert lib.next_batch(8, 32, 1.0, 2.0, 8, 1e-8) == 32  # not falling
    assert lib.next_batch(8, 32, 1.0, 1.0, 8, 1e-8) == 32
    assert lib.next_batch(6, 6, 1.0, 0.5, 8, 1e-8) == 6
