"""Resident runs of more than 1,280 sub-circuits of up to 32 ports, sixteen to a
workgroup, waves between them through LDS: the oracle's iterates, and the sweeps, checks
and result of a launch per sweep (timing = 1 takes that path).

Tolerances: FP64 iterates 1e-11 of max |x| (dot products of at most n_s = 64 terms, over
contracting sweeps); FP32 the bits of the launch per sweep, which rounds alike.
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


# one past the line and a workgroup of one sub-circuit (1,281 = 61 x 21), a ragged last
# row, whole workgroups (1,296), one port a sub-circuit up to all 32, one node each
GRIDS = [((122, 42), (2, 2)), ((287, 290), (8, 8)), ((108, 108), (3, 3)), ((1, 4000), (1, 3)), ((60, 50), (1, 1))]


@pytest.mark.parametrize("dims,block", GRIDS)
def test_iterates(torch, dims, block):
    w = workloads.make(2, nrhs=1, dims=dims, block=block)
    assert w.part.max() + 1 > 1280
    torn = oracle.tear_wires(w.A, w.part, w.Z)
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, 1))
    for sweep in range(1, 8):
        u, a = sw.sweep(torn.src @ w.b.T, a)
        if sweep not in (2, 7):
            continue
        s = vtm().Solver(w.A, w.part, w.Z, check_every=sweep, max_sweeps=sweep, adaptive_checks=False)
        assert resident(s)
        x = torch.empty((1, w.n), dtype=torch.float64, device="cuda")
        with pytest.raises(vtm().VTMError) as ei:
            s.solve(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
        assert ei.value.name == "VTM_E_MAXITER" and resident(s)
        s.close()
        ref = (torn.out @ u).T
        assert np.abs(x.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("dims,block", [((160, 170), (4, 4)), GRIDS[1]])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_same_sweeps_and_checks_as_a_launch_per_sweep(torch, dims, block, precision):
    w = workloads.make(2, nrhs=1, dims=dims, block=block)
    b = torch.as_tensor(w.b, device="cuda")
    got = []
    for timing in (0, 1):
        s = vtm().Solver(w.A, w.part, w.Z, timing=timing, precision=precision)
        for _ in range(2):
            x, rep = s.solve(b, w.tol)
        assert resident(s)
        got.append((x.cpu().numpy(), rep))
        s.close()
    (x0, r0), (x1, r1) = got
    assert (r0.sweeps, r0.outer, r0.checks) == (r1.sweeps, r1.outer, r1.checks)
    assert np.array_equal(r0.history_sweeps, r1.history_sweeps)
    if precision == "fp64":
        assert np.abs(x0 - x1).max() <= 1e-11 * np.abs(x1).max()
    else:
        assert np.array_equal(x0, x1)


@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_a_wait_that_runs_out_falls_back(torch, precision):
    """Every wait bounded to one try: the solve is done again with a launch per sweep."""
    w = workloads.make(2, nrhs=1, dims=(287, 290), block=(8, 8))
    b = torch.as_tensor(w.b, device="cuda")
    s = vtm().Solver(w.A, w.part, w.Z, precision=precision)
    ref, r0 = s.solve(b, w.tol)
    assert resident(s, 0)
    x, rep = s.solve(b, w.tol)
    assert not resident(s, 0)
    assert (rep.sweeps, rep.checks) == (r0.sweeps, r0.checks)
    assert np.abs((x - ref).cpu().numpy()).max() <= 1e-9 * np.abs(ref.cpu().numpy()).max()
