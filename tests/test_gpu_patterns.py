"""The pattern form of the packed layout (constant values per offset and
slice) against the oracle, bit for bit, and where it must not be taken."""
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


def _banded(n, offsets, values, keep=None, seed=3):
    """Rows i with entries at i + offsets (inside the matrix), each kept with
    probability ``keep``; the diagonal (if listed) always."""
    rng = np.random.default_rng(seed)
    cols, vals, rows = [], [], []
    i = np.arange(n, dtype=np.int64)
    for o, v in zip(offsets, values):
        m = (i + o >= 0) & (i + o < n)
        if keep is not None and o != 0:
            m &= rng.random(n) < keep
        rows.append(i[m])
        cols.append(i[m] + o)
        vals.append(np.full(int(m.sum()), v))
    rows, cols, vals = map(np.concatenate, (rows, cols, vals))
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    return rp, cols[order].astype(np.int32), vals[order]


def _is_pattern(A):
    # any other form stores at least the values
    return A.packed_bytes() < 8 * A.nnz


CASES = {
    # name: (matrix, pattern form taken)
    "one row": (lambda: _banded(1, [0], [4.0]), True),
    "last slice of one row": (lambda: _banded(65, [-1, 0, 1], [-1.0, 4.0, -2.0]), True),
    "8 positions": (lambda: _banded(1000, range(-4, 4), np.arange(8) - 10.5), True),
    "9 positions": (lambda: _banded(1000, range(-4, 5), np.arange(9) + 0.25), True),
    "10 positions": (lambda: _banded(1000, range(-5, 5), np.arange(10) + 0.25), True),
    "19 positions, far": (lambda: _banded(4100, np.arange(-9, 10) * 201, np.arange(19) - 30.5), True),
    "32 positions": (lambda: _banded(700, range(-16, 16), np.arange(32) + 1.0), True),
    "33 positions": (lambda: _banded(700, range(-16, 17), np.arange(33) + 1.0), False),
    "no diagonal, all below": (lambda: _banded(500, [-130, -70, -3], [1.0, 2.0, 3.0]), True),
    "all above, empty last rows": (lambda: _banded(500, [2, 65, 200], [1.0, -2.0, 0.5]), True),
    "holes: a slice's list is longer than its rows": (
        lambda: _banded(3000, range(-6, 7), np.arange(13) + 0.5, keep=0.4), True),
    "poisson 40x8x4": (lambda: inputs.poisson7_csr(40, 8, 4), True),
    "27 points 21x13x9": (lambda: inputs.stencil27_csr(21, 13, 9), True),
    "upwind 64x9x5": (lambda: inputs.convdiff7_csr(64, 9, 5), True),
}


@pytest.mark.parametrize("name", CASES)
def test_spmv(name):
    make, pattern = CASES[name]
    Acsr = make()
    n = Acsr[0].size - 1
    A = its().CSRMatrix.from_numpy(*Acsr, validate=False, pack=True, max_fill=8.0)
    if n > 64:
        assert _is_pattern(A) == pattern
    x = inputs.uniform_vector(n, 4)
    assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), oracle.spmv(Acsr, x))


def test_one_value_or_more_patterns_than_the_table_holds():
    rp, col, val = inputs.poisson7_csr(40, 8, 4)
    k = int(rp[700])
    val[k] = np.nextafter(val[k], 0.0)  # one entry differs in its last bit
    # 8300 slices, no two alike
    many = _banded(64 * 8300, [-1, 0, 1], [-1.0, 4.0, -1.0], keep=0.7)
    for Acsr in ((rp, col, val), many):
        A = its().CSRMatrix.from_numpy(*Acsr, validate=False, pack=True, max_fill=8.0)
        assert not _is_pattern(A)
        x = inputs.uniform_vector(Acsr[0].size - 1, 4)
        assert np.array_equal(its().spmv(A, dev(x)).cpu().numpy(), oracle.spmv(Acsr, x))


@pytest.mark.parametrize("values", ["constant", "varying"])
@pytest.mark.parametrize("method", ["cg", "cgnb", "bicgstab", "jacobi", "sgs"])
def test_methods(method, values):
    # 26x9x7 with holes: masked slices, and no box of grid points
    Acsr = inputs.poisson7_csr(26, 9, 7)
    rp, col, val = Acsr
    drop = np.zeros(col.size, bool)
    rows = np.repeat(np.arange(rp.size - 1), np.diff(rp))
    for i in (400, 401, 900):  # symmetric holes
        for j in (i + 1, i + 26):
            drop |= ((rows == i) & (col == j)) | ((rows == j) & (col == i))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows[~drop], minlength=rp.size - 1))]).astype(np.int64)
    col, val = col[~drop], val[~drop].copy()
    if values == "varying":
        val *= 1.0 + 0.125 * np.cos(np.minimum(rows[~drop], col) + 2.0 * np.maximum(rows[~drop], col))
    Acsr = (rp, col, val)
    A = its().CSRMatrix.from_numpy(*Acsr, pack=True)
    assert _is_pattern(A) == (values == "constant")
    n = rp.size - 1
    b = oracle.spmv(Acsr, inputs.uniform_vector(n, 2))
    kw = dict(rtol=0.0, max_iter=4)
    if method == "sgs":
        colors = inputs.redblack_colors(26, 9, 7)
        A.set_colors(colors, 2)
        ref, rr = oracle.sgs(Acsr, colors, 2, b, **kw)
    else:
        ref, rr = getattr(oracle, method)(Acsr, b, **kw)
    x, info = its().solve(A, dev(b), method=method, **kw)
    assert info.iters == rr.iters == 4 and np.array_equal(x.cpu().numpy(), ref)
    if method in ("cg", "cgnb", "bicgstab"):
        x, info = its().solve(A, dev(b), method=method, persistent=True, **kw)
        assert np.array_equal(x.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_refinement(dtype):
    # values that FP16 rounds; a grid whose slices straddle its lines
    Acsr = inputs.stencil_csr(23, 11, 9, [-0.7, -0.9, -1.1, 6.3, -1.1, -0.9, -0.7])
    n = Acsr[0].size - 1
    A = its().CSRMatrix.from_numpy(*Acsr, lowp=(dtype,), pack=True)
    assert _is_pattern(A)
    b = oracle.spmv(Acsr, inputs.uniform_vector(n, 2))
    low = Acsr[2].astype({"f32": np.float32, "f16": np.float16}[dtype]).astype(np.float32)
    ref, rr = oracle.ir_cg(Acsr, low, b, rtol=1e-10, max_iter=500)
    x, info = its().solve(A, dev(b), method="cg", inner_dtype=dtype, rtol=1e-10, max_iter=500)
    assert info.iters == rr.iters and info.inner_iters == rr.inner_iters
    assert np.array_equal(x.cpu().numpy(), ref)
