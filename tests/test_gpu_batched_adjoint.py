"""FP64 adjoints of an unsymmetric A with many right-hand sides, port to port on transposed
operators: the oracle's iterates on A^T, and the sweeps of the full form.

Tolerance: dot products of at most n_s = 512 terms, n_s 2^-53 = 5.7e-14 each, over
contracting sweeps: 1e-11 of max |x|.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


# whole and ragged blocks of up to three ports a node, operators of less than a tile and
# of many; a whole column block, a remainder and several blocks
@pytest.mark.parametrize("dims,block", [((8, 8, 8), (4, 4, 4)), ((9, 11, 10), (3, 4, 5)), ((16, 9, 17), (8, 8, 8))])
@pytest.mark.parametrize("nrhs", [16, 21, 64])
def test_iterates(torch, dims, block, nrhs):
    import paper_0910_0663_amd as vtm
    w = workloads.make(3, nrhs=nrhs, dims=dims, block=block)
    torn = oracle.tear_wires(w.A.T.tocsr(), w.part, w.Z)
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, nrhs))
    for k in range(1, 6):
        u, a = sw.sweep(torn.src @ w.b.T, a)
        if k not in (2, 5):
            continue
        s = vtm.Solver(w.A, w.part, w.Z, nrhs_max=nrhs, check_every=k, max_sweeps=k, adaptive_checks=False, timing=1)
        x = torch.empty((nrhs, w.n), dtype=torch.float64, device="cuda")
        with pytest.raises(vtm.VTMError) as ei:
            s.solve_adjoint(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
        assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.pp_launches == k - 1
        s.close()
        ref = (torn.out @ u).T
        assert np.abs(x.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()


def test_same_sweeps_as_the_full_form_and_after_a_refresh(torch):
    import paper_0910_0663_amd as vtm
    w = workloads.make(3, nrhs=16, dims=(16, 15, 17), block=(8, 8, 8))
    b = torch.as_tensor(w.b, device="cuda")
    got = []
    for form in ("auto", "full"):
        s = vtm.Solver(w.A, w.part, w.Z, nrhs_max=16, **({} if form == "auto" else dict(local_form="full")))
        x, r = s.solve_adjoint(b, w.tol)
        s.refresh(2.0 * w.A.data, Z=0.5 * w.Z)
        x2, r2 = s.solve_adjoint(b, w.tol)
        got.append((x.cpu().numpy(), r.sweeps, x2.cpu().numpy(), r2.sweeps))
        s.close()
    (x, n, x2, n2), (y, m, y2, m2) = got
    assert (n, n2) == (m, m2) and n == n2
    assert np.abs(x - y).max() <= 1e-11 * np.abs(y).max()
    assert np.abs(x2 - y2).max() <= 1e-11 * np.abs(y2).max()
