"""Solves of a million rows and more that stop early launch few iterations in
vain, and the batches of a loop leave the iterates as they are."""
import numpy as np
import pytest

from paper_2305_05988_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

G = (104, 104, 104)  # 1,124,864 points


def its():
    import paper_2305_05988_amd as m
    return m


@pytest.mark.parametrize("method,points,per", [("cg", 7, 1), ("cgnb", 7, 1), ("bicgstab", 7, 1), ("jacobi", 7, 1),
                                               ("sgs", 27, 15)])
@pytest.mark.parametrize("k", [1, 5])
def test_launches(k, method, points, per):
    A = its().StencilMatrix(*G, inputs.POISSON7 if points == 7 else inputs.STENCIL27)
    b = its().spmv(A, torch.from_numpy(inputs.uniform_vector(A.n, 3)).cuda())
    x, info = its().solve(A, b, method=method, rtol=0.0, max_iter=k)
    rtol = info.rel_res * (1.0 + 1e-9)
    y, short = its().solve(A, b, method=method, rtol=rtol, profile=1)
    assert short.status == "ok" and short.iters == k and torch.equal(x, y)
    # class 0: the iteration's first pass, or every sweep of a colour
    assert 0 < short.kernel_launches[0] <= 9 * per


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("method", ["cg", "cgnb", "bicgstab", "jacobi", "sgs"])
def test_batches_do_not_show(method, graph):
    """Stops in a first, a second and a grown batch, at the tolerance and at the
    cap (an odd one, and one just past a batch)."""
    A = its().StencilMatrix(*G, inputs.POISSON7)
    b = its().spmv(A, torch.from_numpy(inputs.uniform_vector(A.n, 3)).cuda())
    for k in (3, 8, 13, 41, 67):
        x, info = its().solve(A, b, method=method, rtol=0.0, max_iter=k, check_every=1)
        for _ in range(2):
            y, one = its().solve(A, b, method=method, rtol=0.0, max_iter=k, graph=graph)
            assert one.iters == info.iters and torch.equal(x, y)
        y, one = its().solve(A, b, method=method, rtol=info.rel_res * (1.0 + 1e-9), graph=graph)
        assert one.status == "ok" and one.iters <= k
        if one.iters == k:
            assert torch.equal(x, y)
