"""Full sweeps of a few large sub-circuits in FP64, whose rows are spread over
workgroups and whose columns over their wavefronts: the oracle's iterates.

Tolerance: dot products of at most n_s = 1,600 terms, n_s 2^-53 = 1.8e-13 a sweep, over
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


# 65 nodes (one row past a workgroup's), an odd count (a last column outside the groups of
# two), fewer column chunks than wavefronts (72 nodes), many more (1,600); ragged blocks and
# sub-circuits of one row; one and several sweeps, of every row and of the port rows alone
@pytest.mark.parametrize("dims,block", [
    ((13, 15), (13, 5)), ((27, 21), (9, 9)), ((24, 25), (8, 9)), ((33, 64), (33, 31)), ((80, 85), (40, 40)),
])
@pytest.mark.parametrize("form", ["full", "port"])
def test_iterates(torch, dims, block, form):
    import paper_0910_0663_amd as vtm
    w = workloads.make(2, dims=dims, block=block)
    torn = oracle.tear_wires(w.A, w.part, w.Z)
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, 1))
    for k in range(1, 5):
        u, a = sw.sweep(torn.src @ w.b.T, a)
        if k == 3:
            continue
        s = vtm.Solver(w.A, w.part, w.Z, check_every=k, max_sweeps=k, adaptive_checks=False, local_form=form)
        x = torch.empty((1, w.n), dtype=torch.float64, device="cuda")
        with pytest.raises(vtm.VTMError) as ei:
            s.solve(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
        assert ei.value.name == "VTM_E_MAXITER"
        s.close()
        ref = (torn.out @ u).T
        err = np.abs(x.cpu().numpy() - ref).max()
        assert err <= 1e-11 * np.abs(ref).max(), (k, err)
