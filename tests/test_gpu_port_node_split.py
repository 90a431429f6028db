"""FP64 sweeps of dense port-node operators, 64 rows a workgroup and their columns over its
wavefronts, one launch per sweep (timing = 1 takes that path): the oracle's iterates.

Tolerance: dot products of at most n_s = 4,225 terms, n_s 2^-53 = 4.7e-13 each, over
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


# port nodes of the largest sub-circuit: 65 (a last row block of one row, an odd column),
# 81, 113, 129 (one row past two blocks), 218, 260 and 271, with one to three ports a node;
# several and ragged sub-circuits, fewer column pairs than a wavefront's first loads and
# several times as many; both directions of an unsymmetric A
@pytest.mark.parametrize("cfg,dims,block,k", [
    (2, (66, 66), (33, 33), 65), (2, (82, 82), (41, 41), 81), (2, (114, 114), (57, 57), 113),
    (2, (130, 130), (65, 65), 129), (3, (20, 20, 20), (10, 10, 10), 271), (3, (17, 16, 18), (8, 8, 8), 260),
    (3, (21, 22, 20), (7, 7, 7), 218),
])
def test_iterates(torch, cfg, dims, block, k):
    import paper_0910_0663_amd as vtm
    w = workloads.make(cfg, nrhs=1, dims=dims, block=block)
    wires = oracle.tear_wires(w.A, w.part, w.Z).meta["wires"]
    nodes = np.unique(np.concatenate([wires[0], wires[1]]))
    assert np.bincount(w.part[nodes]).max() == k
    for adjoint in (False, True):
        torn = oracle.tear_wires(w.A.T.tocsr() if adjoint else w.A, w.part, w.Z)
        sw = oracle.Sweeper(torn)
        a = np.zeros((2, torn.n_lines, 1))
        for sweep in range(1, 8):
            u, a = sw.sweep(torn.src @ w.b.T, a)
            if sweep not in (2, 7):
                continue
            s = vtm.Solver(w.A, w.part, w.Z, check_every=sweep, max_sweeps=sweep, adaptive_checks=False, timing=1)
            x = torch.empty((1, w.n), dtype=torch.float64, device="cuda")
            with pytest.raises(vtm.VTMError) as ei:
                (s.solve_adjoint if adjoint else s.solve)(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
            assert ei.value.name == "VTM_E_MAXITER"
            s.close()
            ref = (torn.out @ u).T
            err = np.abs(x.cpu().numpy() - ref).max()
            assert err <= 1e-11 * np.abs(ref).max(), (adjoint, sweep, err)
