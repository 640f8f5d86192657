"""Passes that sum the partials of the pass before them themselves (at most
1024 blocks and partials) and passes behind a finishing kernel: both sides of
the line, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2305_05988_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def its():
    import paper_2305_05988_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _line(n):
    """Tridiagonal (-1, 2.5, -1.25): as many rows as wanted, two colours."""
    i = np.arange(n, dtype=np.int64)
    cols = np.concatenate([i - 1, i, i + 1])
    rows = np.concatenate([i, i, i])
    vals = np.concatenate([np.full(n, -1.0), np.full(n, 2.5), np.full(n, -1.25)])
    keep = (cols >= 0) & (cols < n)
    order = np.lexsort((cols[keep], rows[keep]))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=n))]).astype(np.int64)
    return rp, cols[keep][order].astype(np.int32), vals[keep][order]


ROWS = 256


# one block; a grid on both sides of 1024 blocks; the update passes' 1024 blocks
# behind a pass of more; graphs at two sizes
SIZES = [(n, False) for n in (1, 255, 1024 * ROWS, 1024 * ROWS + 1, 2048 * ROWS + 77)]
SIZES += [(255, True), (1024 * ROWS + 1, True)]


@pytest.mark.parametrize("n,graph", SIZES)
@pytest.mark.parametrize("method", ["cg", "cgnb", "bicgstab", "jacobi", "sgs"])
@pytest.mark.parametrize("pack", [False, True])
def test_both_sides(pack, method, n, graph):
    Acsr = _line(n)
    A = its().CSRMatrix.from_numpy(*Acsr, pack=pack, max_fill=4.0)
    b = inputs.uniform_vector(n, 3)
    kw = dict(rtol=0.0, max_iter=5)
    if method == "sgs":
        colors = (np.arange(n) % 2).astype(np.uint8)
        A.set_colors(colors, 2)
        ref, rr = oracle.sgs(Acsr, colors, 2, b, **kw)
    else:
        ref, rr = getattr(oracle, method)(Acsr, b, **kw)
    for _ in range(3 if graph else 1):
        x, info = its().solve(A, dev(b), method=method, graph=graph, **kw)
        assert info.iters == rr.iters
        assert np.array_equal(x.cpu().numpy(), ref)
        assert abs(info.rel_res - rr.rel_res) <= 1e-12 * rr.rel_res


# the persistent kernels of matrix-free stencils: rows up to 131,072 points,
# bricks beyond; one row per thread up to 256 blocks (65,536 rows) and several
@pytest.mark.parametrize("method", ["cg", "cgnb", "bicgstab"])
@pytest.mark.parametrize("g", [(1, 1, 1), (64, 32, 32), (64, 33, 32), (64, 32, 64), (64, 33, 63)])
@pytest.mark.parametrize("points", [7, 27])
def test_persistent_stencils(points, g, method):
    coef = {7: inputs.convdiff7() if method == "bicgstab" else inputs.POISSON7, 27: inputs.STENCIL27}[points]
    Acsr = inputs.stencil_csr(*g, coef)
    b = inputs.uniform_vector(Acsr[0].size - 1, 3)
    ref, rr = getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=4)
    x, info = its().solve(its().StencilMatrix(*g, coef), dev(b), method=method, rtol=0.0, max_iter=4, persistent=True)
    assert info.iters == rr.iters and np.array_equal(x.cpu().numpy(), ref)
