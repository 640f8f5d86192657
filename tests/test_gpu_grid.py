"""The plane sweep of constant stencils (grids of at least 360,448 points; two
points per thread below 5 * 2^20, four from there on) and of variable
coefficients against the oracle, bit for bit: ragged tiles, lines cut into uneven tiles, thin grids, short last chunks,
and packed matrices that are a stencil on a grid or just not one."""
import numpy as np
import pytest

import oracle
from paper_2305_05988_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

COEF = {7: [-1.0, -1.25, -0.75, 6.5, -0.75, -1.25, -1.0],
        27: [-1.0 + 0.01 * abs(q - 13) for q in range(13)] + [26.5] + [-1.0 + 0.01 * abs(q - 13) for q in range(14, 27)]}
UPWIND = inputs.convdiff7()
# two points per thread: ragged tiles; three tiles a line; lines of 3 points; a
# line of 110 and a line of 111 (the widest tile and past it); a last chunk of
# one plane; two planes; past 128; the smallest.  Four points per thread: ragged;
# thin planes
GRIDS = [(131, 97, 67), (260, 61, 53), (3, 300, 900), (110, 85, 85), (111, 90, 81), (90, 90, 109), (640, 641, 2),
         (129, 128, 128), (64, 64, 88), (181, 173, 170), (64, 17, 4831)]


def its():
    import paper_2305_05988_amd as m
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


_cache = {}


def _system(g, coef):
    """The last system only: some hold tens of millions of entries."""
    key = (g, tuple(coef))
    if key not in _cache:
        _cache.clear()
        Acsr = inputs.stencil_csr(*g, coef)
        x = inputs.uniform_vector(Acsr[0].size - 1, 4)
        _cache[key] = (Acsr, x, oracle.spmv(Acsr, x))
    return _cache[key]


def _operator(Acsr, g, coef, form):
    if form == "free":
        return its().StencilMatrix(*g, coef)
    A = its().CSRMatrix.from_numpy(*Acsr, pack=True, max_fill=4.0)
    assert A.packed_bytes() == 8 * len(coef)  # found to be a stencil on a grid
    return A


def _check(A, b, ref, rr, method, k, **kw):
    x, info = its().solve(A, dev(b), method=method, rtol=0.0, max_iter=k, **kw)
    assert info.iters == rr.iters == k and info.restarts == rr.restarts
    # where the method itself overflows (CG-NB on extreme k) the oracle holds the same NaN
    assert np.array_equal(x.cpu().numpy(), ref, equal_nan=True)
    assert abs(info.rel_res - rr.rel_res) <= 1e-12 * rr.rel_res


@pytest.mark.parametrize("g", GRIDS)
def test_spmv_and_krylov_7(g):
    Acsr, x, b = _system(g, COEF[7])
    cg, bi = oracle.cg(Acsr, b, rtol=0.0, max_iter=3), None
    for form in ("free", "packed"):
        A = _operator(Acsr, g, COEF[7], form)
        assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
        _check(A, b, *cg, "cg", 3)
        _check(A, b, *cg, "cg", 3, graph=True)
    jac = oracle.jacobi(Acsr, b, rtol=0.0, max_iter=3)
    _check(A, b, *jac, "jacobi", 3)


@pytest.mark.parametrize("g", [GRIDS[0], GRIDS[4], GRIDS[6], GRIDS[7], GRIDS[9]])
def test_27(g):
    Acsr, x, b = _system(g, COEF[27])
    A = _operator(Acsr, g, COEF[27], "packed" if g == GRIDS[0] else "free")
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
    _check(A, b, *oracle.cg(Acsr, b, rtol=0.0, max_iter=2), "cg", 2)
    _check(A, b, *oracle.jacobi(Acsr, b, rtol=0.0, max_iter=2), "jacobi", 2)
    if g == GRIDS[0]:  # eight colours: the residual test of an iteration
        S = its().StencilMatrix(*g, COEF[27])
        _check(S, b, *oracle.sgs(Acsr, inputs.octant_colors(*g), 8, b, rtol=0.0, max_iter=1), "sgs", 1)


# with and without restarts (every iteration whose cosine is below 0.9)
@pytest.mark.parametrize("restart_tol", [1e-5, 0.9])
@pytest.mark.parametrize("g", [GRIDS[0], GRIDS[9]])
def test_bicgstab(g, restart_tol):
    Acsr, _, b = _system(g, UPWIND)
    ref = oracle.bicgstab(Acsr, b, rtol=0.0, max_iter=5, restart_tol=restart_tol)
    if restart_tol > 0.5:
        assert ref[1].restarts >= 2
    for form in ("free", "packed"):
        _check(_operator(Acsr, g, UPWIND, form), b, *ref, "bicgstab", 5, restart_tol=restart_tol)
    At = its().StencilMatrix(*g, tuple(reversed(UPWIND)))
    _check(At, b, *ref, "bicgstab", 5, restart_tol=restart_tol, transpose=True)


def test_cgnb():
    Acsr, _, b = _system(GRIDS[0], COEF[7])
    for form in ("free", "packed"):
        _check(_operator(Acsr, GRIDS[0], COEF[7], form), b, *oracle.cgnb(Acsr, b, rtol=0.0, max_iter=4), "cgnb", 4)


@pytest.mark.parametrize("points,g", [(7, GRIDS[1]), (7, GRIDS[9]), (27, GRIDS[0])])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_refinement(dtype, points, g):
    Acsr, _, b = _system(g, COEF[points])
    low = Acsr[2].astype({"f32": np.float32, "f16": np.float16}[dtype]).astype(np.float32)
    kw = dict(rtol=1e-30, max_iter=7, inner_rtol=1e-1)
    ref, rr = oracle.ir_cg(Acsr, low, b, **kw)
    A = its().CSRMatrix.from_numpy(*Acsr, lowp=(dtype,), pack=True, max_fill=4.0)
    assert A.packed_bytes(dtype) == 4 * points
    x, info = its().solve(A, dev(b), method="cg", inner_dtype=dtype, **kw)
    assert info.iters == rr.iters and info.inner_iters == rr.inner_iters
    assert np.array_equal(x.cpu().numpy(), ref)


@pytest.mark.parametrize("what", ["value", "entry", "wrapped"])
def test_almost_a_grid(what):
    g = (131, 97, 67)
    rp, col, val = (a.copy() for a in _system(g, COEF[7])[0])
    n = rp.size - 1
    if what == "value":  # constant in its slice, another value elsewhere
        val[int(rp[64 * 5000]):int(rp[64 * 5001])] *= 0.5
    else:
        rows = np.repeat(np.arange(n), np.diff(rp))
        if what == "entry":  # one missing coupling
            drop = (rows == 500000) & (col == 500001)
            keep = ~drop
            rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=n))]).astype(rp.dtype)
            col, val = col[keep], val[keep]
        else:  # couplings across the ends of the lines
            i = np.arange(n)
            d = np.array([-131 * 97, -131, -1, 0, 1, 131, 131 * 97])
            c = i[:, None] + d
            keep = (c >= 0) & (c < n)
            rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64)
            col, val = c[keep].astype(np.int32), np.broadcast_to(np.array(COEF[7]), c.shape)[keep].copy()
    A = its().CSRMatrix.from_numpy(rp, col, val, pack=True, max_fill=4.0)
    assert A.packed_bytes() > 56
    x = inputs.uniform_vector(n, 4)
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), oracle.spmv((rp, col, val), x))


# "far": some k outside the range of
# the plain quotient (2^-250 to 2^250), so some planes take the general one
@pytest.mark.parametrize("g,far", [((131, 97, 67), False), ((90, 90, 109), True), ((640, 641, 2), False),
                                   ((165, 141, 140), False)])
def test_variable_coefficients(g, far):
    n = g[0] * g[1] * g[2]
    rng = np.random.default_rng(5)
    k = np.exp(rng.standard_normal(n))
    if far:
        k[rng.integers(0, n, 40)] *= 1e-80
        k[rng.integers(0, n, 40)] *= 1e85
    Acsr = oracle.varcoef_csr(*g, k)
    A = its().VarCoefMatrix(*g, dev(k))
    x = inputs.uniform_vector(n, 4)
    b = oracle.spmv(Acsr, x)
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), b)
    if g[2] == 140:
        _check(A, b, *oracle.cg(Acsr, b, rtol=0.0, max_iter=3), "cg", 3)
        return
    for method in ("cg", "cgnb", "bicgstab", "jacobi"):
        ref, rr = getattr(oracle, method)(Acsr, b, rtol=0.0, max_iter=3)
        if rr.iters < 3:  # extreme k: BiCGStab's own products overflow
            assert far and method == "bicgstab"
            continue
        _check(A, b, ref, rr, method, 3)


# odd and even lines; two and four points per thread; the colours swapped (no
# plane sweep, the colours' own rows)
@pytest.mark.parametrize("g", [GRIDS[0], GRIDS[1], GRIDS[6], GRIDS[9]])
def test_red_black(g):
    Acsr, _, b = _system(g, COEF[7])
    colors = inputs.redblack_colors(*g)
    ref = oracle.sgs(Acsr, colors, 2, b, rtol=0.0, max_iter=3)
    S = its().StencilMatrix(*g, COEF[7])
    A = _operator(Acsr, g, COEF[7], "packed")
    A.set_colors(colors, 2)
    for M in (S, A):
        _check(M, b, *ref, "sgs", 3)
        _check(M, b, *ref, "sgs", 3, graph=True)
        # a solve that stops at a tolerance returns the tested iterate
        rtol = 0.5 * (ref[1].rel_res + oracle.sgs(Acsr, colors, 2, b, rtol=0.0, max_iter=2)[1].rel_res)
        x, info = its().solve(M, dev(b), method="sgs", rtol=rtol, max_iter=50)
        assert info.status == "ok" and info.iters == 3 and np.array_equal(x.cpu().numpy(), ref[0])
    if g == GRIDS[0]:
        swapped = (1 - colors).astype(np.uint8)
        A.set_colors(swapped, 2)
        _check(A, b, *oracle.sgs(Acsr, swapped, 2, b, rtol=0.0, max_iter=2), "sgs", 2)
