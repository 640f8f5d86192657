"""The work that users of this library have it do, as cases to be timed.

Each case is one call (or one forward and backward call) of the package's
public entry points on a seeded problem whose solution is known: x* is drawn
from the seed and b = A x* is formed with plain torch, so `exact` can say how
far an answer is from the solution itself.

Families (`kind`):

  spmv     y = A x
  solve    its.solve to a relative residual, every method and precision
  smooth   its.solve stopped after a fixed number of sweeps (Jacobi and
           symmetric Gauss-Seidel as smoothers)
  adjoint  its.csr_solve forward and backward: gradients of the right-hand
           side and of the stored values (a transposed solve)
  diffuse  its.diffusion_solve forward and backward: gradients of the
           right-hand side and of the per-cell coefficients
  batch    its.Batch.solve, many systems with several right-hand sides

Operators (`op`): the 7-point Poisson, 27-point and upwind convection-diffusion
operators of inputs.py ("poisson", "p27", "upwind"), the variable-coefficient
diffusion ("varying", k = exp(g), g ~ N(0, 1) per cell) and an irregular
matrix whose row lengths and columns are random ("irregular").  `form`: how
the user holds the operator: "csr", "packed" (CSR packed by the library) or
"free" (matrix-free).
"""
from __future__ import annotations

import math

import torch

import paper_2305_05988_amd as its
from paper_2305_05988_amd import inputs

COEF = {"poisson": inputs.POISSON7, "p27": inputs.STENCIL27, "upwind": inputs.convdiff7(10.0)}


def listed():
    return [
        # the smallest solves: latency counts, one cooperative launch
        dict(name="cg_free_32_persistent", kind="solve", op="poisson", form="free", nx=32, ny=32, nz=32,
             method="cg", inner="f64", rtol=1e-8, persistent=True),
        # a small ragged system solved with the default options
        dict(name="cg_packed_45x38x41", kind="solve", op="poisson", form="packed", nx=45, ny=38, nz=41,
             method="cg", inner="f64", rtol=1e-8, persistent=False),
        # the headline workload of bench.py
        dict(name="cg_packed_256", kind="solve", op="poisson", form="packed", nx=256, ny=256, nz=256,
             method="cg", inner="f64", rtol=1e-8, persistent=False),
        # a matrix whose values differ from row to row, on a ragged grid
        dict(name="cg_varying_packed_131x118x107", kind="solve", op="varying", form="packed", nx=131, ny=118,
             nz=107, method="cg", inner="f64", rtol=1e-8, persistent=False),
        # a matrix-free solve that streams from HBM
        dict(name="cg_free_256x240x200", kind="solve", op="poisson", form="free", nx=256, ny=240, nz=200,
             method="cg", inner="f64", rtol=1e-8, persistent=False),
        # mixed-precision refinement on the dense stencil
        dict(name="refine_f16_p27_192", kind="solve", op="p27", form="packed", nx=192, ny=192, nz=192,
             method="cg", inner="f16", rtol=1e-8, persistent=False),
        # nonsymmetric solve and its adjoint, with the gradient of the values
        dict(name="adjoint_upwind_160x144x150", kind="adjoint", op="upwind", form="packed", nx=160, ny=144,
             nz=150, method="bicgstab", rtol=1e-10),
        # smoothing sweeps on the dense stencil and on a ragged 7-point grid
        dict(name="jacobi_p27_packed_120x110x96", kind="smooth", op="p27", form="packed", nx=120, ny=110, nz=96,
             method="jacobi", sweeps=40),
        dict(name="sgs_packed_192x160x170", kind="smooth", op="poisson", form="packed", nx=192, ny=160, nz=170,
             method="sgs", sweeps=30),
        # the differentiable solve of bench.py
        dict(name="diffusion_grad_128", kind="diffuse", op="varying", form="free", nx=128, ny=128, nz=128,
             method="cg", rtol=1e-10),
        # uneven systems with eight right-hand sides each
        dict(name="batch_96x8", kind="batch", systems=96, rhs=8, lo=16, hi=64, rtol=1e-8),
        # one product with an irregular matrix as given
        dict(name="spmv_irregular_700k", kind="spmv", op="irregular", form="csr", rows=700_000, mean=20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi, most):
    while True:
        s = [_log(rng, lo, hi) for _ in range(3)]
        if s[0] * s[1] * s[2] <= most:
            return dict(nx=s[0], ny=s[1], nz=s[2])


def draw(rng):
    kind = rng.choice(["spmv", "solve", "solve", "solve", "solve", "solve", "smooth", "adjoint", "diffuse", "batch"])
    if kind == "spmv":
        op = rng.choice(["irregular", "poisson", "p27", "varying"])
        if op == "irregular":
            return dict(kind=kind, op=op, form="csr", rows=_log(rng, 2000, 1_000_000), mean=rng.randint(5, 40))
        form = rng.choice(["csr", "packed", "free"]) if op != "varying" else rng.choice(["packed", "free"])
        return dict(kind=kind, op=op, form=form, **_sides(rng, 12, 250, 8_000_000))
    if kind == "solve":
        what = rng.choice(["small", "krylov", "krylov", "refine"])
        if what == "small":
            op = rng.choice(["poisson", "poisson", "upwind"])
            method = "bicgstab" if op == "upwind" else rng.choice(["cg", "cgnb", "bicgstab"])
            return dict(kind=kind, op=op, form=rng.choice(["packed", "free"]), method=method, inner="f64", rtol=1e-8,
                        persistent=rng.random() < 0.5, **_sides(rng, 14, 56, 100_000))
        if what == "refine":
            return dict(kind=kind, op=rng.choice(["poisson", "p27"]), form=rng.choice(["packed", "packed", "csr"]),
                        method="cg", inner=rng.choice(["f32", "f16"]), rtol=1e-8, persistent=False,
                        **_sides(rng, 40, 220, 6_000_000))
        op = rng.choice(["poisson", "p27", "upwind", "varying"])
        method = "bicgstab" if op == "upwind" else rng.choice(["cg", "cg", "cgnb", "bicgstab"])
        return dict(kind=kind, op=op, form=rng.choice(["packed", "packed", "free", "csr"]), method=method,
                    inner="f64", rtol=1e-8, persistent=False,
                    **_sides(rng, 40, 240, 2_000_000 if op == "varying" else 8_000_000))
    if kind == "smooth":
        op = rng.choice(["poisson", "p27"])
        return dict(kind=kind, op=op, form=rng.choice(["packed", "packed", "free", "csr"]),
                    method=rng.choice(["jacobi", "sgs"]), sweeps=rng.randint(4, 50),
                    **_sides(rng, 30, 220, 4_000_000))
    if kind == "adjoint":
        return dict(kind=kind, op="upwind", form=rng.choice(["packed", "csr"]), method="bicgstab", rtol=1e-10,
                    **_sides(rng, 30, 200, 4_000_000))
    if kind == "diffuse":
        return dict(kind=kind, op="varying", form="free", method="cg", rtol=1e-10, **_sides(rng, 20, 140, 1_500_000))
    return dict(kind=kind, systems=_log(rng, 4, 96), rhs=rng.choice([1, 2, 4, 8]), lo=16, hi=rng.randint(24, 64),
                rtol=1e-8)


# ------------------------------------------------------------------ problems

def _gen(seed, device="cuda"):
    return torch.Generator(device=device).manual_seed(int(seed))


def _uniform(n, g):
    return torch.rand(n, dtype=torch.float64, device="cuda", generator=g) * 2.0 - 1.0


def _offsets(case):
    return inputs.OFFSETS27 if case["op"] == "p27" else inputs.OFFSETS7


def _window(n, d):
    """Slices (of the rows, of their neighbours) along one axis for offset d."""
    return slice(max(0, -d), n - max(0, d)), slice(max(0, d), n - max(0, -d))


def _pairs(dims, offset):
    nx, ny, nz = dims
    dk, dj, di = offset
    (zr, zn), (yr, yn), (xr, xn) = _window(nz, dk), _window(ny, dj), _window(nx, di)
    return (zr, yr, xr), (zn, yn, xn)


def _dims(case):
    return case["nx"], case["ny"], case["nz"]


def _apply(coef, offsets, dims, x, transpose=False):
    """A x of a constant stencil."""
    v = x.view(dims[2], dims[1], dims[0])
    y = torch.zeros_like(v)
    for c, o in zip(coef, offsets):
        rows, nbrs = _pairs(dims, o if not transpose else tuple(-d for d in o))
        y[rows] += c * v[nbrs]
    return y.view(-1)


FACES = tuple(o for o in inputs.OFFSETS7 if o != (0, 0, 0))


def _faces(dims, k):
    """The six face coefficients of each cell (harmonic means; the cell's own
    coefficient at the boundary), in the order of FACES."""
    v = k.view(dims[2], dims[1], dims[0])
    out = []
    for o in FACES:
        rows, nbrs = _pairs(dims, o)
        f = v.clone()
        f[rows] = 2.0 * v[rows] * v[nbrs] / (v[rows] + v[nbrs])
        out.append(f)
    return out


def _apply_varying(dims, k, x):
    v = x.view(dims[2], dims[1], dims[0])
    y = torch.zeros_like(v)
    for o, f in zip(FACES, _faces(dims, k)):
        rows, nbrs = _pairs(dims, o)
        y += f * v
        y[rows] -= f[rows] * v[nbrs]
    return y.view(-1)


def _csr(case, k=None):
    """CSR arrays (row_ptr int32, col int32, val float64) on the GPU."""
    nx, ny, nz = dims = _dims(case)
    n = nx * ny * nz
    offsets = _offsets(case)
    count = torch.zeros(nz, ny, nx, dtype=torch.int32, device="cuda")
    for o in offsets:
        count[_pairs(dims, o)[0]] += 1
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(count.view(-1), 0, out=rp[1:])
    nnz = int(rp[-1])
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    val = torch.empty(nnz, dtype=torch.float64, device="cuda")
    row = torch.arange(n, device="cuda").view(nz, ny, nx)
    at = rp[:-1].clone().view(nz, ny, nx)
    faces = dict(zip(FACES, _faces(dims, k))) if k is not None else None
    for i, o in enumerate(offsets):
        rows, nbrs = _pairs(dims, o)
        p = at[rows].reshape(-1)
        col[p] = row[nbrs].reshape(-1).to(torch.int32)
        if faces is None:
            val[p] = float(COEF[case["op"]][i])
        else:
            val[p] = (-faces[o][rows]).reshape(-1) if o in faces else sum(faces.values()).reshape(-1)
        at[rows] += 1
    return rp.to(torch.int32), col, val


def _irregular(case, g):
    """Rows of 0 to 2 mean entries at random columns near and far."""
    n, mean = case["rows"], case["mean"]
    length = torch.randint(0, 2 * mean + 1, (n,), device="cuda", generator=g)
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), length)
    near = row + torch.randint(-1000, 1001, (row.numel(),), device="cuda", generator=g)
    far = torch.randint(0, n, (row.numel(),), device="cuda", generator=g)
    pick = torch.rand(row.numel(), device="cuda", generator=g) < 0.8
    key = torch.unique(row * n + torch.where(pick, near, far).remainder(n))
    row, col = key // n, (key % n).to(torch.int32)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(row, minlength=n), 0, out=rp[1:])
    return rp.to(torch.int32), col, _uniform(col.numel(), g)


def _batch_dims(case):
    """The grid sides of a batch: the same for every seed."""
    g = _gen(7, "cpu")
    return torch.randint(case["lo"], case["hi"] + 1, (case["systems"], 3), generator=g).tolist()


def _problem(case, seed):
    """What the seed decides: coefficients and solutions."""
    g = _gen(seed)
    if case["kind"] == "batch":
        cells = sum(a * b * c for a, b, c in _batch_dims(case))
        return dict(k=torch.exp(torch.randn(cells, dtype=torch.float64, device="cuda", generator=g)),
                    x=_uniform(cells * case["rhs"], g))
    if case["op"] == "irregular":
        rp, col, val = _irregular(case, g)
        return dict(rp=rp, col=col, val=val, x=_uniform(case["rows"], g))
    n = case["nx"] * case["ny"] * case["nz"]
    p = dict(x=_uniform(n, g))
    if case["kind"] in ("adjoint", "diffuse"):
        p["lam"] = _uniform(n, g)
    if case["op"] == "varying":
        p["k"] = torch.exp(torch.randn(n, dtype=torch.float64, device="cuda", generator=g))
    return p


def _times(case, p, x, transpose=False):
    if case["op"] == "varying":
        return _apply_varying(_dims(case), p["k"], x)
    return _apply(COEF[case["op"]], _offsets(case), _dims(case), x, transpose)


def _operator(case, p):
    nx, ny, nz = _dims(case)
    if case["form"] == "free":
        if case["op"] == "varying":
            return its.VarCoefMatrix(nx, ny, nz, p["k"])
        return its.StencilMatrix(nx, ny, nz, COEF[case["op"]])
    rp, col, val = _csr(case, p.get("k"))
    inner = case.get("inner", "f64")
    low = its.cast_values(val, inner) if inner != "f64" else None
    A = its.CSRMatrix(rp, col, val, val32=low if inner == "f32" else None, val16=low if inner == "f16" else None)
    if case["form"] == "packed":
        A.pack()
    if case.get("method") == "sgs":
        i = torch.arange(nx, device="cuda").view(1, 1, nx)
        j = torch.arange(ny, device="cuda").view(1, ny, 1)
        k = torch.arange(nz, device="cuda").view(nz, 1, 1)
        color = (i + j + k) % 2 if case["op"] != "p27" else i % 2 + 2 * (j % 2) + 4 * (k % 2)
        A.set_colors(color.to(torch.uint8).reshape(-1).contiguous(), 2 if case["op"] != "p27" else 8)
    return A


def prepare(case, seed):
    p = _problem(case, seed)
    kind = case["kind"]
    if kind == "batch":
        dims = _batch_dims(case)
        b, at = torch.empty_like(p["x"]).view(-1, case["rhs"]), 0
        xs = p["x"].view(-1, case["rhs"])
        for d in dims:
            n = d[0] * d[1] * d[2]
            for r in range(case["rhs"]):
                b[at:at + n, r] = _apply_varying(d, p["k"][at:at + n], xs[at:at + n, r].contiguous())
            at += n
        B = its.Batch(dims, p["k"], case["rhs"])
        return dict(kind=kind, B=B, b=b.view(-1), rtol=case["rtol"])
    if kind == "spmv":
        A = its.CSRMatrix(p["rp"], p["col"], p["val"]) if case["op"] == "irregular" else _operator(case, p)
        return dict(kind=kind, A=A, x=p["x"], y=torch.empty_like(p["x"]))
    b = _times(case, p, p["x"])
    if kind == "diffuse":
        return dict(kind=kind, k=p["k"].requires_grad_(), b=b.requires_grad_(), gx=_times(case, p, p["lam"]),
                    shape=_dims(case), opts=dict(method=case["method"], rtol=case["rtol"]))
    A = _operator(case, p)
    if kind == "adjoint":
        A.build_transpose()
        A.val.requires_grad_()
        return dict(kind=kind, A=A, b=b.requires_grad_(), gx=_times(case, p, p["lam"], transpose=True),
                    opts=dict(method=case["method"], rtol=case["rtol"]))
    if kind == "smooth":
        opts = dict(method=case["method"], rtol=1e-14, max_iter=case["sweeps"])
    else:
        opts = dict(method=case["method"], rtol=case["rtol"], inner_dtype=case["inner"],
                    persistent=case["persistent"])
    return dict(kind=kind, A=A, b=b, opts=opts, ws=torch.empty(its.api.workspace_bytes(A, **opts), dtype=torch.uint8,
                                                               device="cuda"))


def run(state):
    kind = state["kind"]
    if kind == "spmv":
        return its.spmv(state["A"], state["x"], state["y"])
    if kind == "batch":
        x, info = state["B"].solve(state["b"], rtol=state["rtol"])
        return {"x": x, "iters": info.iters}
    if kind == "diffuse":
        x = its.diffusion_solve(state["k"], state["b"], state["shape"], **state["opts"])
        dk, db = torch.autograd.grad(x, (state["k"], state["b"]), state["gx"])
        return {"x": x, "dk": dk, "db": db}
    if kind == "adjoint":
        x = its.csr_solve(state["A"], state["b"], **state["opts"])
        dval, db = torch.autograd.grad(x, (state["A"].val, state["b"]), state["gx"])
        return {"x": x, "dval": dval, "db": db}
    x, info = its.solve(state["A"], state["b"], workspace=state["ws"], **state["opts"])
    return {"x": x, "iters": info.iters}


def exact(case, seed):
    """The solution the inputs were made from, its gradients, or the iterate
    of plain torch sweeps.  A solve to a tolerance is as far from it as its
    tolerance allows."""
    p = _problem(case, seed)
    kind, x = case["kind"], p["x"]
    if kind == "batch" or kind == "solve":
        return {"x": x, "iters": None}
    if kind == "spmv":
        if case["op"] != "irregular":
            return _times(case, p, x)
        A = torch.sparse_csr_tensor(p["rp"].long(), p["col"].long(), p["val"], (case["rows"], case["rows"]))
        return A @ x
    if kind == "adjoint":
        rp, col, _ = _csr(case)
        row = torch.repeat_interleave(torch.arange(x.numel(), device="cuda"), (rp[1:] - rp[:-1]).long())
        return {"x": x, "dval": -p["lam"][row] * x[col.long()], "db": p["lam"]}
    if kind == "diffuse":
        dims = _dims(case)
        shape = (dims[2], dims[1], dims[0])
        k, xv, lam = p["k"].view(shape), x.view(shape), p["lam"].view(shape)
        dk = torch.zeros_like(k)
        for o in FACES:
            rows, nbrs = _pairs(dims, o)
            t = lam * xv  # boundary faces
            w = 2.0 * k[nbrs] ** 2 / (k[rows] + k[nbrs]) ** 2
            t[rows] = w * (lam[rows] - lam[nbrs]) * (xv[rows] - xv[nbrs])
            dk -= t
        return {"x": x, "dk": dk.view(-1), "db": p["lam"]}
    # the smoothers, started from 0
    dims, offsets, coef = _dims(case), _offsets(case), COEF[case["op"]]
    shape = (dims[2], dims[1], dims[0])
    centre = dict(zip(offsets, coef))[(0, 0, 0)]
    b = _times(case, p, x)
    v = torch.zeros_like(b)

    def relaxed():
        return v + (b - _apply(coef, offsets, dims, v)) / centre

    if case["method"] == "jacobi":
        for _ in range(case["sweeps"]):
            v = relaxed()
        return {"x": v, "iters": case["sweeps"]}
    grid = torch.meshgrid(*(torch.arange(m, device="cuda") for m in shape), indexing="ij")
    color = (sum(grid) % 2 if case["op"] != "p27" else grid[2] % 2 + 2 * (grid[1] % 2) + 4 * (grid[0] % 2)).view(-1)
    order = list(range(2 if case["op"] != "p27" else 8))
    for _ in range(case["sweeps"]):
        for c in order + order[::-1]:
            v = torch.where(color == c, relaxed(), v)
    return {"x": v, "iters": case["sweeps"]}


# ---------------------------------------------------------------------- work

def _iterations(case):
    """About how many iterations the solve takes: counts of measured solves,
    fitted over the mean side of the grid."""
    nx, ny, nz = _dims(case)
    side = (nx * ny * nz) ** (1.0 / 3.0)
    if case["op"] == "varying":
        return 6.6 * side * (math.log10(case["rtol"]) / -8.0) * (0.65 if case["method"] == "bicgstab" else 1.0)
    if case["op"] == "upwind":
        return 1.9 * side
    cg = 107.0 * (side / 32.0) ** 0.68 * (0.6 if case["op"] == "p27" else 1.0)
    return cg * (0.65 if case["method"] == "bicgstab" else 1.0)


def work(case):
    """Bytes: per pass over the operator, 8 bytes for every value that differs
    from row to row (a constant stencil holds none, a variable-coefficient
    operator one per cell matrix-free and one per entry as a matrix), and the
    vectors.  The scalar products cut an iteration of CG into two passes: the
    first reads r and p, the second reads and writes them and moves x: 7
    vectors.  BiCGStab: three passes, 17 vectors.  A Jacobi sweep: x, b in and
    x out; a symmetric Gauss-Seidel sweep: twice that.  The refinement's inner
    vectors are 4 bytes wide."""
    kind = case["kind"]
    if kind == "batch":
        cells = sum(a * b * c for a, b, c in _batch_dims(case))
        n = cells * case["rhs"]
        iters = 6.6 * (cells / case["systems"]) ** (1.0 / 3.0)
        return {"bytes": iters * 8.0 * (7 * n + 2 * cells), "flops": iters * 23.0 * n}
    if case["op"] == "irregular":
        nnz = case["rows"] * case["mean"]
        return {"bytes": 12.0 * nnz + 20.0 * case["rows"], "flops": 2.0 * nnz}
    nx, ny, nz = _dims(case)
    n = nx * ny * nz
    per_row = 27 if case["op"] == "p27" else 7
    matrix = 0 if case["op"] != "varying" else 8 * n * (1 if case["form"] == "free" else per_row)
    if kind == "spmv":
        return {"bytes": matrix + 16.0 * n, "flops": 2.0 * per_row * n}
    if kind == "smooth":
        twice = 1 if case["method"] == "jacobi" else 2
        return {"bytes": case["sweeps"] * twice * (matrix + 24.0 * n),
                "flops": case["sweeps"] * twice * (2.0 * per_row + 4) * n}
    v = 8 if case.get("inner", "f64") == "f64" else 4
    iters = _iterations(case)
    if case["method"] == "bicgstab":
        one = {"bytes": iters * (2 * matrix + 17.0 * v * n), "flops": iters * (4.0 * per_row + 20) * n}
    else:
        one = {"bytes": iters * (matrix + 7.0 * v * n), "flops": iters * (2.0 * per_row + 10) * n}
    if kind in ("adjoint", "diffuse"):  # forward and adjoint solve, then the gradient
        extra = (8 * per_row if kind == "adjoint" else 8) * n + 24.0 * n
        return {"bytes": 2 * one["bytes"] + extra, "flops": 2 * one["flops"] + 20.0 * n}
    return one
