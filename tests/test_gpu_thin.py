"""Thin grids of more than 360,448 points, which the plane sweep leaves to the
packed rows and the bricks, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2305_05988_amd import inputs

from . import grid_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def its():
    import paper_2305_05988_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(A, b, ref, rr, method, k):
    x, info = its().solve(A, dev(b), method=method, rtol=0.0, max_iter=k)
    assert info.iters == rr.iters == k and np.array_equal(x.cpu().numpy(), ref)
    assert abs(info.rel_res - rr.rel_res) <= 1e-12 * rr.rel_res


# a duct in z, packed and matrix-free (its bricks several planes thick); a line
# of points along each axis; the sweep of two points per thread on 5 * 2^20
# points and more
@pytest.mark.parametrize("g", [(8, 8, 6000), (1, 1, 370000), (370000, 1, 1), (16, 16, 20500)])
def test_thin(g):
    print(f"thin grid {g}", flush=True)
    coef = [-1.0, -1.25, -0.75, 6.5, -0.75, -1.25, -1.0]
    Acsr = inputs.stencil_csr(*g, coef)
    x = inputs.uniform_vector(Acsr[0].size - 1, 4)
    b = oracle.spmv(Acsr, x)
    forms = [its().StencilMatrix(*g, coef)]
    if min(g) > 1:
        P = its().CSRMatrix.from_numpy(*Acsr, pack=True, max_fill=4.0)
        assert (P.packed_bytes() == 56) == grid_plan.takes(7, g, packed=True)
        forms.append(P)
        P.set_colors(inputs.redblack_colors(*g), 2)
    refs = {m: getattr(oracle, m)(Acsr, b, rtol=0.0, max_iter=3) for m in ("cg", "jacobi", "bicgstab")}
    refs["sgs"] = oracle.sgs(Acsr, inputs.redblack_colors(*g), 2, b, rtol=0.0, max_iter=3)
    for A in forms:
        assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
        for m, ref in refs.items():
            _check(A, b, *ref, m, 3)


def test_thin_variable_coefficients():
    g = (300, 3, 900)
    assert not grid_plan.takes(1, g)
    n = g[0] * g[1] * g[2]
    k = np.exp(np.random.default_rng(5).standard_normal(n))
    Acsr = oracle.varcoef_csr(*g, k)
    b = oracle.spmv(Acsr, inputs.uniform_vector(n, 4))
    _check(its().VarCoefMatrix(*g, dev(k)), b, *oracle.cg(Acsr, b, rtol=0.0, max_iter=3), "cg", 3)
