"""Resident runs of sub-circuits one to a compute unit (FP64 of more than 128 ports, FP32):
the oracle's iterates, and the sweeps, checks and result of a launch per sweep
(timing = 1 takes that path).

Tolerance: dot products of at most n_s = 4,225 terms, n_s 2^-53 = 4.7e-13 each, over
contracting sweeps: 1e-11 of max |x|.
"""
import ctypes as C

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


def vtm():
    import paper_0910_0663_amd as v
    return v


def resident(s, ticks=400_000_000):
    f = vtm().lib().vtm_testing_wait_ticks
    f.argtypes, f.restype = [C.c_void_p, C.c_uint64], C.c_int
    return bool(f(s._h, ticks))


# most port nodes and ports of a sub-circuit: two to five row groups of 64 rows, odd and
# even counts, one to three ports a node, ragged sub-circuits, operators in registers, in
# LDS and streamed; more than 320 nodes or 512 ports stay with a launch per sweep
@pytest.mark.parametrize("cfg,dims,block,nodes,ports,res", [
    (2, (102, 102), (34, 34), 132, 136, True), (3, (15, 15, 15), (5, 5, 5), 98, 150, True),
    (2, (130, 130), (65, 65), 129, 130, True), (3, (20, 20, 20), (10, 10, 10), 271, 300, True),
    (3, (18, 17, 19), (6, 6, 6), 152, 216, True), (3, (21, 22, 20), (7, 7, 7), 218, 294, True),
    (3, (17, 16, 18), (8, 8, 8), 260, 320, True), (3, (24, 24, 24), (8, 8, 8), 296, 384, True),
    (3, (27, 27, 18), (9, 9, 9), 337, 405, False),
])
def test_iterates(torch, cfg, dims, block, nodes, ports, res):
    w = workloads.make(cfg, nrhs=1, dims=dims, block=block)
    i, j, _ = oracle.tear_wires(w.A, w.part, w.Z).meta["wires"]
    assert np.bincount(w.part[np.unique(np.concatenate([i, j]))]).max() == nodes
    assert np.bincount(np.concatenate([w.part[i], w.part[j]])).max() == ports
    for adjoint in (False, True):
        torn = oracle.tear_wires(w.A.T.tocsr() if adjoint else w.A, w.part, w.Z)
        sw = oracle.Sweeper(torn)
        a = np.zeros((2, torn.n_lines, 1))
        for sweep in range(1, 8):
            u, a = sw.sweep(torn.src @ w.b.T, a)
            if sweep not in (2, 7):
                continue
            s = vtm().Solver(w.A, w.part, w.Z, check_every=sweep, max_sweeps=sweep, adaptive_checks=False)
            assert resident(s) == res
            x = torch.empty((1, w.n), dtype=torch.float64, device="cuda")
            with pytest.raises(vtm().VTMError) as ei:
                (s.solve_adjoint if adjoint else s.solve)(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
            assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.sweeps == sweep
            assert resident(s) == res   # no wait ran out
            s.close()
            ref = (torn.out @ u).T
            err = np.abs(x.cpu().numpy() - ref).max()
            assert err <= 1e-11 * np.abs(ref).max(), (adjoint, sweep, err)


@pytest.mark.parametrize("cfg,dims,block", [(3, (24, 24, 24), (8, 8, 8)), (2, (150, 120), (50, 40))])
def test_same_sweeps_and_checks_as_a_launch_per_sweep(torch, cfg, dims, block):
    w = workloads.make(cfg, nrhs=1, dims=dims, block=block)
    b = torch.as_tensor(w.b, device="cuda")
    got = []
    for timing in (0, 1):
        s = vtm().Solver(w.A, w.part, w.Z, timing=timing)
        for _ in range(2):
            x, rep = s.solve(b, w.tol)
        assert resident(s)
        got.append((x.cpu().numpy(), rep))
        s.close()
    (x0, r0), (x1, r1) = got
    assert (r0.sweeps, r0.checks) == (r1.sweeps, r1.checks)
    assert np.array_equal(r0.history_sweeps, r1.history_sweeps)
    assert np.abs(x0 - x1).max() <= 1e-11 * np.abs(x1).max()


# FP32: the bits of a launch per sweep, on operators of two to five row groups, counts of
# every remainder by four, symmetric and not
@pytest.mark.parametrize("cfg,dims,block", [
    (2, (72, 72), (24, 24)), (2, (130, 130), (65, 65)), (3, (9, 10, 12), (3, 3, 3)), (3, (18, 17, 19), (6, 6, 6)),
    (3, (21, 22, 20), (7, 7, 7)), (3, (20, 20, 20), (10, 10, 10)), (3, (17, 16, 18), (8, 8, 8)),
    (3, (24, 24, 24), (8, 8, 8)), (4, (180, 170), None),
])
def test_fp32_same_as_a_launch_per_sweep(torch, cfg, dims, block):
    w = workloads.make(cfg, nrhs=1, dims=dims, **({} if block is None else dict(block=block)))
    b = torch.as_tensor(w.b, device="cuda")
    for adjoint in (False, True):
        got = []
        for timing in (0, 1):
            s = vtm().Solver(w.A, w.part, w.Z, timing=timing, precision="fp32_refine")
            x, rep = (s.solve_adjoint if adjoint else s.solve)(b, w.tol)
            assert resident(s)
            got.append((x.cpu().numpy(), rep))
            s.close()
        (x0, r0), (x1, r1) = got
        assert (r0.sweeps, r0.outer, r0.checks) == (r1.sweeps, r1.outer, r1.checks)
        assert np.array_equal(x0, x1)


def test_a_wait_that_runs_out_falls_back(torch):
    """Every wait bounded to one try: the solve is done again with a launch per sweep."""
    w = workloads.make(3, nrhs=1, dims=(24, 24, 24), block=(8, 8, 8))
    b = torch.as_tensor(w.b, device="cuda")
    s = vtm().Solver(w.A, w.part, w.Z)
    ref, r0 = s.solve(b, w.tol)
    assert resident(s, 0)
    x, rep = s.solve(b, w.tol)
    assert not resident(s, 0)
    assert (rep.sweeps, rep.checks) == (r0.sweeps, r0.checks)
    assert np.abs((x - ref).cpu().numpy()).max() <= 1e-9 * np.abs(ref.cpu().numpy()).max()
