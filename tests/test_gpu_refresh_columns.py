"""vtm_refresh on handles of several columns: new values reach every copy of the operators
that their sweeps use, so that solves equal those of a fresh handle, bit for bit."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


# packed and dense port-node operators as tiles (transposed ones for the adjoint of an
# unsymmetric A), the dense port operator, batched tiles of an unsymmetric A
@pytest.mark.parametrize("cfg,kw,prec,nrhs,form", [
    (2, dict(dims=(40, 33)), "fp64", 3, "port"), (1, dict(dims=(49, 64)), "fp32_refine", 7, "port"),
    (3, dict(dims=(16, 16, 9)), "fp64", 7, "port"), (3, dict(dims=(16, 16, 9)), "fp32_refine", 3, "port"),
    (2, dict(dims=(40, 33)), "fp64", 3, "port_dense"), (3, dict(dims=(16, 16, 9)), "fp64", 16, "port"),
])
def test_refresh_equals_fresh_setup(torch, cfg, kw, prec, nrhs, form):
    import paper_0910_0663_amd as vtm
    w = workloads.make(cfg, nrhs=nrhs, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    # the same pattern: every entry by 1.25, and more to ground at each node
    A = (1.25 * w.A + sp.diags(np.random.default_rng(3).uniform(0.0, 0.1, w.n))).tocsr()
    A.sort_indices()
    assert np.array_equal(A.indices, w.A.tocsr().indices)
    opt = dict(precision=prec, nrhs_max=nrhs, local_form=form)
    s = vtm.Solver(w.A, w.part, w.Z, **opt)
    s.solve(b, 1e-8)
    s.refresh(A)
    t = vtm.Solver(A, w.part, w.Z, **opt)
    for one, two in ((s.solve, t.solve), (s.solve_adjoint, t.solve_adjoint)):
        (x, rx), (y, ry) = one(b, 1e-8), two(b, 1e-8)
        assert torch.equal(x, y) and (rx.sweeps, rx.outer, rx.checks) == (ry.sweeps, ry.outer, ry.checks)
    s.close()
    t.close()
