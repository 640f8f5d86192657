"""Refinement with a coefficient beyond the range of the low precision that no
row has: a grid one point wide in x."""
import numpy as np
import pytest

import oracle
from paper_2305_05988_amd import inputs

from . import grid_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_unused_coefficient_overflows_f16():
    import paper_2305_05988_amd as its
    g = (1, 700, 701)
    assert grid_plan.takes(7, g)
    coef = [-1.0, -1.25, 1e6, 6.5, 1e6, -1.25, -1.0]
    Acsr = inputs.stencil_csr(*g, coef)
    b = oracle.spmv(Acsr, inputs.uniform_vector(Acsr[0].size - 1, 2))
    low = Acsr[2].astype(np.float16).astype(np.float32)
    assert np.isfinite(low).all()
    kw = dict(rtol=1e-10, max_iter=500)
    ref, rr = oracle.ir_cg(Acsr, low, b, **kw)
    x, info = its.solve(its.StencilMatrix(*g, coef), torch.from_numpy(b).cuda(), method="cg", inner_dtype="f16", **kw)
    assert info.status == "ok" and info.iters == rr.iters and info.inner_iters == rr.inner_iters
    assert np.array_equal(x.cpu().numpy(), ref)
