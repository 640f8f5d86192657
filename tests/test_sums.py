"""The serial sum of block partials (csrc/dd.hpp, compiled for the host)
against exact rational arithmetic."""
import ctypes as C
from fractions import Fraction

import numpy as np
import pytest

from . import grid_plan

U = Fraction(1, 2 ** 53)


@pytest.fixture(scope="module")
def lib():
    return grid_plan.build("""
#define __device__
#define __forceinline__ inline
#include "dd.hpp"
extern "C" void dd_sum2(const its::DD *a, const its::DD *b, int first, int step, int count, its::DD *out) {
  const its::DD *src[2] = {a, b};
  its::DD v[2];
  its::dd_sum<2>(src, first, step, count, v);
  out[0] = v[0];
  out[1] = v[1];
}
""")


def _sum(lib, pairs, first=0, step=1):
    a = [np.ascontiguousarray(p) for p in pairs]
    out = np.empty((2, 2))
    lib.dd_sum2(*(C.c_void_p(p.ctypes.data) for p in a), first, step, len(a[0]), C.c_void_p(out.ctypes.data))
    return [Fraction(h) + Fraction(l) for h, l in out]


def _bound(pairs):
    """Exact sum, and the bound of as many accurate additions: each adds at most
    3 u^2 / (1 - 4 u) of its result (Joldes, Muller and Popescu), which differs from
    the exact partial sum by no more than the error so far."""
    s, total = Fraction(0), 0.0
    for h, l in pairs:
        s += Fraction(h) + Fraction(l)
        total += abs(float(s))
    return s, 3 * U * U * Fraction(total) * Fraction(1001, 1000)


@pytest.mark.parametrize("seed", range(4))
def test_error_follows_the_sum(lib, seed):
    # high parts that cancel in pairs over low parts of one sign
    rng = np.random.default_rng(seed)
    n = 4096
    pairs = []
    for sign in (1.0, -1.0):
        hi = 1.0 + rng.random(n)
        hi[1::2] = -hi[::2]
        lo = sign * np.spacing(np.abs(hi)) * (0.25 + 0.25 * rng.random(n))
        pairs.append(np.stack([hi, lo], 1))
    for got, p in zip(_sum(lib, pairs), pairs):
        exact, bound = _bound(p)
        assert abs(got - exact) <= bound


def test_partials_of_a_thread(lib):
    # powers of two: every sum is exact, so the indices that were added show
    count = 37
    p = np.stack([2.0 ** np.arange(count), np.zeros(count)], 1)
    for first, step in ((0, 1), (3, 8), (36, 8), (37, 8), (5, 256)):
        want = sum(2 ** j for j in range(first, count, step))
        assert _sum(lib, [p, p], first, step) == [want, want]
