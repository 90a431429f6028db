"""A solve repeated on one handle, through vtm_solve and vtm_solve_noalloc, gives the same
bits and report whatever ran on the handle before (vtm_solve_noalloc promises those of
vtm_solve): resident runs of every shape, after odd and even numbers of sweeps.
"""
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


# packed operators of up to 32 ports in twos and sixteens, 64, 96 and 128 ports; a compute
# unit each in registers, LDS and streamed from the L2
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine"])
@pytest.mark.parametrize("cfg,kw", [
    (2, dict(dims=(40, 40))), (2, dict(dims=(368, 240))), (1, dict(dims=(33, 64))), (2, dict(dims=(72, 72), block=(24, 24))),
    (2, dict(dims=(96, 96), block=(32, 32))), (3, dict(dims=(15, 15, 15), block=(5, 5, 5))),
    (3, dict(dims=(21, 22, 20), block=(7, 7, 7))), (3, dict(dims=(24, 24, 24), block=(8, 8, 8))),
])
def test_same_bits(torch, cfg, kw, prec):
    import paper_0910_0663_amd as vtm
    w = workloads.make(cfg, nrhs=1, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    s = vtm.Solver(w.A, w.part, w.Z, precision=prec)
    x, rep = s.solve(b, w.tol)
    # other tolerances between: runs of other lengths leave the exchange words elsewhere
    for k, tol in enumerate((w.tol, 1e-2, w.tol, 3e-3, w.tol, 1e-4, w.tol, 1e-5, w.tol, 1e-6, w.tol, w.tol)):
        y, r = (s.solve_noalloc if k % 2 else s.solve)(b, tol)
        if tol == w.tol:
            assert torch.equal(x, y) and (r.sweeps, r.outer, r.checks) == (rep.sweeps, rep.outer, rep.checks)
    s.close()
