"""The plane sweep on grids of 2^23 points and more: tiles of whole 128-byte
lines, and matrix-free CG left to the bricks, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2305_05988_amd import inputs

from . import grid_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

COEF = [-1.0, -1.25, -0.75, 6.5, -0.75, -1.25, -1.0]


def its():
    import paper_2305_05988_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# tiles wider than what is left of a line; one tile a line, wider than the line;
# CG by bricks (its first member a sweep's residual)
@pytest.mark.parametrize("g,W,cg", [((272, 272, 115), 48, True), ((72, 90, 1300), 80, True), ((261, 259, 250), None, False)])
def test_large(g, W, cg):
    print(f"large grid {g}", flush=True)
    s = grid_plan.shape(7, g)
    assert s.points == 4 and (W is None or s.W == W) and grid_plan.takes_cg(7, g) == cg
    Acsr = inputs.stencil_csr(*g, COEF)
    x = inputs.uniform_vector(Acsr[0].size - 1, 4)
    b = oracle.spmv(Acsr, x)
    A = its().StencilMatrix(*g, COEF)
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
    for method in ("cg",) if not cg else ("cg", "jacobi", "bicgstab"):
        ref, rr = getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=3)
        y, info = its().solve(A, dev(b), method=method, rtol=0.0, max_iter=3)
        assert info.iters == rr.iters and np.array_equal(y.cpu().numpy(), ref)
        assert abs(info.rel_res - rr.rel_res) <= 1e-12 * rr.rel_res
        # a solve that stops after an odd count of iterations, and the residual of its x
        y2, one = its().solve(A, dev(b), method=method, rtol=info.rel_res * (1 + 1e-9))
        assert one.status == "ok" and one.iters <= 3
        if one.iters < 3:  # the residual need not fall at every iteration
            continue
        assert torch.equal(y, y2)
        assert abs(one.true_rel_res - info.true_rel_res) <= 1e-12 * info.true_rel_res
