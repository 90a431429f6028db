"""FP64 sweeps of packed port-node operators of up to 8 port nodes and just above, two
sub-circuits a wavefront, one launch per sweep (timing = 1 takes that path): the oracle's
iterates.

Tolerance: dot products of at most n_s = 20 terms, n_s 2^-53 = 2.2e-15 each, over
contracting sweeps: 1e-11 of max |x| as for larger sub-circuits.
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


# port nodes of the largest sub-circuit: 1 to 8, 9 and 10, with one to four ports a node; ragged
# ones beside them, and an odd number of sub-circuits (the last one alone)
@pytest.mark.parametrize("dims,block,nodes,odd", [
    ((9, 7), (1, 1), 1, True), ((10, 6), (2, 1), 2, False), ((9, 11), (3, 1), 3, True), ((17, 13), (2, 2), 4, True),
    ((8, 15), (1, 5), 5, False), ((9, 9), (3, 2), 6, True), ((21, 3), (7, 1), 7, True), ((20, 16), (3, 3), 8, False),
    ((24, 2), (8, 1), 8, False), ((12, 15), (4, 3), 10, True), ((27, 3), (9, 1), 9, True),
])
@pytest.mark.parametrize("per_wire", [False, True])
def test_iterates(torch, dims, block, nodes, odd, per_wire):
    import paper_0910_0663_amd as vtm
    w = workloads.make(2, dims=dims, block=block)
    i, j, _ = oracle.tear_wires(w.A, w.part, w.Z).meta["wires"]
    assert np.bincount(w.part[np.unique(np.concatenate([i, j]))]).max() == nodes
    assert (w.part.max() + 1) % 2 == int(odd)
    Z = w.Z * np.random.default_rng(1).uniform(0.7, 1.4, i.size) if per_wire else w.Z
    torn = oracle.tear_wires(w.A, w.part, Z)
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, 1))
    for k in range(1, 8):
        u, a = sw.sweep(torn.src @ w.b.T, a)
        if k not in (2, 7):
            continue
        ref = (torn.out @ u).T
        s = vtm.Solver(w.A, w.part, Z, check_every=k, max_sweeps=k, adaptive_checks=False, timing=1)
        x = torch.empty(w.b.shape, dtype=torch.float64, device="cuda")
        with pytest.raises(vtm.VTMError) as ei:
            s.solve(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
        assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.sweeps == k
        s.close()
        assert np.abs(x.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()
