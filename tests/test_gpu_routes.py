"""Kernels that only some sizes and forms reach, each at such a size, against
the oracle bit for bit: the plane sweep on flat grids (more bricks than blocks,
more blocks than the passes sum themselves), wide tiles, transposed and
low-precision operators on it; bricks of several planes; the packed layout with
a value per entry, in every precision, with blocks that walk several tiles; and
passes of more than 4096 blocks."""
import numpy as np
import pytest

import oracle
from paper_2305_05988_amd import inputs

from . import grid_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

COEF = {7: [-1.0, -1.25, -0.75, 6.5, -0.75, -1.25, -1.0],
        27: [-1.0 + 0.01 * abs(q - 13) for q in range(13)] + [26.5] + [-1.0 + 0.01 * abs(q - 13) for q in range(14, 27)]}
UPWIND = list(inputs.convdiff7())
SWAPPED = UPWIND[::-1]


def its():
    import paper_2305_05988_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(A, b, ref, rr, method, k, **kw):
    print(f"routes: {method} {kw}", flush=True)
    x, info = its().solve(A, dev(b), method=method, rtol=0.0, max_iter=k, **kw)
    assert info.iters == rr.iters and info.restarts == rr.restarts
    assert np.array_equal(x.cpu().numpy(), ref)
    assert abs(info.rel_res - rr.rel_res) <= 1e-12 * rr.rel_res


def _lowp(val, dtype):
    return val.astype({"f32": np.float32, "f16": np.float16}[dtype]).astype(np.float32)


def _check_refinement(A, Acsr, b, dtype):
    kw = dict(rtol=1e-30, max_iter=7, inner_rtol=1e-1)
    ref, rr = oracle.ir_cg(Acsr, _lowp(Acsr[2], dtype), b, **kw)
    x, info = its().solve(A, dev(b), method="cg", inner_dtype=dtype, **kw)
    assert info.iters == rr.iters and info.inner_iters == rr.inner_iters
    assert np.array_equal(x.cpu().numpy(), ref)


# ------------------------------------------------------------- plane sweep

# more than 1024 bricks (finishing kernels between the passes) and more than
# 4096 (a block takes several bricks), of two points per thread and of four
@pytest.mark.parametrize("npts,g,points,bricks", [(7, (1000, 1000, 1), 2, (1025, 4096)), (7, (2000, 2000, 1), 2, (4097, 1 << 20)),
                                                  (27, (2000, 2000, 1), 2, (4097, 1 << 20)),
                                                  (7, (2400, 2400, 1), 4, (4097, 1 << 20))])
def test_flat_grids(npts, g, points, bricks):
    s = grid_plan.shape(npts, g)
    assert grid_plan.takes(npts, g) and s.points == points and bricks[0] <= s.bricks <= bricks[1]
    Acsr = inputs.stencil_csr(*g, COEF[npts])
    x = inputs.uniform_vector(Acsr[0].size - 1, 4)
    b = oracle.spmv(Acsr, x)
    A = its().StencilMatrix(*g, COEF[npts])
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
    for method in ("cg", "jacobi", "cgnb") if npts == 7 else ("cg", "jacobi"):
        _check(A, b, *getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=3), method, 3)
    if npts == 7:
        _check(A, b, *oracle.sgs(Acsr, inputs.redblack_colors(*g), 2, b, rtol=0.0, max_iter=3), "sgs", 3)
        up = inputs.stencil_csr(*g, UPWIND)
        _check(its().StencilMatrix(*g, UPWIND), b, *oracle.bicgstab(up, b, rtol=0.0, max_iter=3), "bicgstab", 3)


# "far": coefficients outside the range of the plain quotient in some bricks
@pytest.mark.parametrize("far", [False, True])
def test_flat_variable_coefficients(far):
    g = (1447, 1448, 3)
    assert grid_plan.takes(1, g) and grid_plan.shape(1, g).bricks > 4096
    n = g[0] * g[1] * g[2]
    rng = np.random.default_rng(5)
    k = np.exp(rng.standard_normal(n))
    if far:
        k[rng.integers(0, n, 40)] *= 1e-80
    Acsr = oracle.varcoef_csr(*g, k)
    b = oracle.spmv(Acsr, inputs.uniform_vector(n, 4))
    A = its().VarCoefMatrix(*g, dev(k))
    for method in ("cg", "jacobi"):
        _check(A, b, *getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=2), method, 2)


@pytest.mark.parametrize("g,points", [((146, 146, 60), 2), ((142, 194, 200), 4)])
def test_tiles_wider_than_a_wave(g, points):
    s = grid_plan.shape(7, g)
    assert grid_plan.takes(7, g, packed=True) and s.W > 64 and s.points == points
    Acsr = inputs.stencil_csr(*g, COEF[7])
    b = oracle.spmv(Acsr, inputs.uniform_vector(Acsr[0].size - 1, 4))
    ref = oracle.cg(Acsr, b, rtol=0.0, max_iter=3)
    _check(its().StencilMatrix(*g, COEF[7]), b, *ref, "cg", 3)
    _check(its().CSRMatrix.from_numpy(*Acsr, pack=True), b, *ref, "cg", 3)


SWEPT = (131, 97, 67)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("transpose", [False, True])
def test_matrix_free_refinement_by_planes(dtype, transpose):
    assert grid_plan.takes(7, SWEPT)
    Acsr = inputs.stencil_csr(*SWEPT, SWAPPED if transpose else UPWIND)
    b = oracle.spmv(Acsr, inputs.uniform_vector(Acsr[0].size - 1, 4))
    kw = dict(rtol=1e-30, max_iter=7, inner_rtol=1e-1)
    ref, rr = oracle.ir_cg(Acsr, _lowp(Acsr[2], dtype), b, **kw)
    x, info = its().solve(its().StencilMatrix(*SWEPT, UPWIND), dev(b), method="cg", inner_dtype=dtype,
                          transpose=transpose, **kw)
    assert info.iters == rr.iters and info.inner_iters == rr.inner_iters
    assert np.array_equal(x.cpu().numpy(), ref)


def test_transposed_by_planes():
    Tcsr = inputs.stencil_csr(*SWEPT, SWAPPED)
    b = oracle.spmv(Tcsr, inputs.uniform_vector(Tcsr[0].size - 1, 4))
    S = its().StencilMatrix(*SWEPT, UPWIND)
    colors = inputs.redblack_colors(*SWEPT)
    _check(S, b, *oracle.sgs(Tcsr, colors, 2, b, rtol=0.0, max_iter=3), "sgs", 3, transpose=True)
    _check(S, b, *oracle.jacobi(Tcsr, b, rtol=0.0, max_iter=3), "jacobi", 3, transpose=True)
    A = its().CSRMatrix.from_numpy(*inputs.stencil_csr(*SWEPT, UPWIND), pack=True)
    assert A.packed_bytes() == 56
    A.build_transpose()
    for graph in (False, True):
        _check(A, b, *oracle.bicgstab(Tcsr, b, rtol=0.0, max_iter=4), "bicgstab", 4, transpose=True, graph=graph)


# ------------------------------------------------------ bricks of several planes

@pytest.mark.parametrize("points", [7, 27])
def test_persistent_stencil_bricks(points):
    g = (130, 64, 100)
    S = its().StencilMatrix(*g, COEF[points])
    assert S.n > 1 << 17 and S.plan[3] > 1
    Acsr = inputs.stencil_csr(*g, COEF[points])
    b = oracle.spmv(Acsr, inputs.uniform_vector(S.n, 4))
    for method in ("cg", "cgnb", "bicgstab"):
        _check(S, b, *getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=3), method, 3, persistent=True)


@pytest.mark.parametrize("g,persistent", [((190, 186, 180), False), ((131, 97, 67), True)])
def test_variable_coefficient_bricks(g, persistent):
    n = g[0] * g[1] * g[2]
    k = np.exp(np.random.default_rng(5).standard_normal(n))
    A = its().VarCoefMatrix(*g, dev(k))
    assert A.plan[3] > 1 and (persistent or not grid_plan.takes(1, g))
    Acsr = oracle.varcoef_csr(*g, k)
    b = oracle.spmv(Acsr, inputs.uniform_vector(n, 4))
    for method in ("cg",) if persistent else ("cg", "jacobi"):
        _check(A, b, *getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=2), method, 2, persistent=persistent)


# ------------------------------------------------- packed, a value per entry

def _varying(g, points):
    rp, col, val = inputs.stencil_csr(*g, COEF[points], *(() if points == 7 else (inputs.OFFSETS27,)))
    rows = np.repeat(np.arange(rp.size - 1), np.diff(rp))
    lo, hi = np.minimum(rows, col), np.maximum(rows, col)
    return rp, col, val * (1.0 + 0.125 * np.cos(lo + 2.0 * hi))


# one slice and a piece; a few tiles; blocks that walk several tiles
@pytest.mark.parametrize("g,points", [((23, 11, 9), 7), ((23, 11, 9), 27), ((5, 5, 3), 7), ((104, 103, 105), 7), ((104, 103, 105), 27)])
def test_packed_values(g, points):
    Acsr = _varying(g, points)
    n = Acsr[0].size - 1
    A = its().CSRMatrix.from_numpy(*Acsr, lowp=("f32", "f16"), pack=True, max_fill=4.0)
    assert A.packed_bytes() >= 8 * A.nnz  # values per entry
    x = inputs.uniform_vector(n, 4)
    b = oracle.spmv(Acsr, x)
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
    for method in ("cg", "cgnb", "bicgstab", "jacobi"):
        _check(A, b, *getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=3), method, 3)
    colors, nc = (inputs.redblack_colors(*g), 2) if points == 7 else (inputs.octant_colors(*g), 8)
    A.set_colors(colors, nc)
    _check(A, b, *oracle.sgs(Acsr, colors, nc, b, rtol=0.0, max_iter=2), "sgs", 2)
    for dtype in ("f32", "f16"):
        _check_refinement(A, Acsr, b, dtype)


# ------------------------------------------------ passes of more than 4096 blocks

@pytest.mark.parametrize("pack", [False, True])
def test_two_levels_of_partials(pack):
    n = 4 * 4096 * 256 + 1000  # more than four tiles for each of 4096 blocks: a block a tile
    i = np.arange(n, dtype=np.int64)
    cols = np.stack([i - 1, i, i + 1], 1)
    vals = np.stack([-1.0 + 0.125 * np.cos(i), np.full(n, 2.5), -1.0 + 0.125 * np.cos(i + 1.0)], 1)
    keep = (cols >= 0) & (cols < n)
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64)
    Acsr = (rp, cols[keep].astype(np.int32), vals[keep])
    A = its().CSRMatrix.from_numpy(*Acsr, pack=pack, max_fill=4.0)
    b = inputs.uniform_vector(n, 3)
    for method in ("cg", "cgnb", "bicgstab", "jacobi"):
        ref = getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=3)
        _check(A, b, *ref, method, 3)
    colors = (i % 2).astype(np.uint8)
    A.set_colors(colors, 2)
    _check(A, b, *oracle.sgs(Acsr, colors, 2, b, rtol=0.0, max_iter=2), "sgs", 2)
