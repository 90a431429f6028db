"""FP64 sweeps of the packed port-node operators, two sub-circuits a wavefront, one
launch per sweep (timing = 1 takes that path): the oracle's iterates.

Tolerance: dot products of at most n_s = 961 terms, n_s 2^-53 = 1.1e-13 each, over
contracting sweeps: 1e-11 of max |x|.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


def solver(w, k):
    import paper_0910_0663_amd as vtm
    return vtm.Solver(w.A, w.part, w.Z, check_every=k, max_sweeps=k, adaptive_checks=False, timing=1)


def run(torch, s, b, adjoint=False):
    import paper_0910_0663_amd as vtm
    x = torch.empty(b.shape, dtype=torch.float64, device="cuda")
    with pytest.raises(vtm.VTMError) as ei:
        (s.solve_adjoint if adjoint else s.solve)(torch.as_tensor(b, device="cuda"), 1e-300, x)
    return ei.value.name, x.cpu().numpy()


# one port a sub-circuit up to all 32 lanes; an odd number of sub-circuits (the last one
# alone), pairs of unequal ones (ragged blocks, random cuts), one and several ports a node
@pytest.mark.parametrize("cfg,dims,block", [
    (2, (2, 6), (2, 1)), (2, (1, 9), (1, 3)), (2, (12, 20), (4, 4)), (2, (24, 24), (8, 8)), (2, (23, 31), (8, 8)),
    (2, (29, 26), (7, 9)), (2, (62, 31), (31, 31)), (2, (16, 48), (16, 16)), (2, (40, 3), (1, 1)),
])
@pytest.mark.parametrize("k", [2, 7])
def test_iterates(torch, cfg, dims, block, k):
    w = workloads.make(cfg, dims=dims, block=block)
    torn = oracle.tear_wires(w.A, w.part, w.Z)
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, 1))
    for _ in range(k):
        u, a = sw.sweep(torn.src @ w.b.T, a)
    ref = (torn.out @ u).T
    s = solver(w, k)
    name, x = run(torch, s, w.b)
    s.close()
    assert name == "VTM_E_MAXITER"
    assert np.abs(x - ref).max() <= 1e-11 * np.abs(ref).max()


def test_what_is_not_finite_stays_in_its_component(torch):
    """Two grids without a branch between them, their sub-circuits in turn along the
    wavefronts: a source that is not a number in one leaves the other's waves alone."""
    w = workloads.make(2, dims=(24, 24), block=(8, 8))
    w.A = sp.block_diag([w.A, w.A]).tocsr()
    w.part = np.concatenate([2 * w.part, 2 * w.part + 1])
    b = np.concatenate([w.b, w.b], axis=1)
    bad = b.copy()
    bad[0, 300] = np.nan
    waves = []
    for v in (b, bad):
        s = solver(w, 6)
        name, _ = run(torch, s, v)
        assert name == ("VTM_E_MAXITER" if v is b else "VTM_E_DIVERGED")
        waves.append(s.get_waves().cpu().numpy().reshape(2, -1))
        s.close()
    assert np.isfinite(waves[0]).all() and not np.isfinite(waves[1][0]).all()
    assert np.array_equal(waves[0][1], waves[1][1])
