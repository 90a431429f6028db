"""Resident runs (all port-to-port sweeps and checks of a one-column solve in one
launch) against the oracle and against a launch per sweep (timing = 1 takes that
path), through the C ABI.

Tolerances: FP64 iterates 1e-11 of max |x| (dot products of at most n_s = 1,089 terms,
n_s 2^-53 = 1.2e-13 each, over contracting sweeps); FP32 iterates 5.5 sqrt(k) u
sqrt((2 + n_s) / 3) 8 of max |x|, u = 2^-24.  The decisions of the checks are compared
through the sweeps at which they fell.
"""
import ctypes as C
import math
import threading

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


def wait_ticks(s, ticks=400_000_000):
    f = vtm().lib().vtm_testing_wait_ticks
    f.argtypes, f.restype = [C.c_void_p, C.c_uint64], C.c_int
    return bool(f(s._h, ticks))


def reference(A, w, k):
    torn = oracle.tear_wires(A, w.part, w.Z)
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, 1))
    for _ in range(k):
        u, a = sw.sweep(torn.src @ w.b.T, a)
    return (torn.out @ u).T


def iterate(torch, w, k, resident, adjoint=False, **kw):
    s = vtm().Solver(w.A, w.part, w.Z, check_every=k, max_sweeps=k, adaptive_checks=False, **kw)
    assert wait_ticks(s) == resident
    x = torch.empty((1, w.n), dtype=torch.float64, device="cuda")
    with pytest.raises(vtm().VTMError) as ei:
        (s.solve_adjoint if adjoint else s.solve)(torch.as_tensor(w.b, device="cuda"), 1e-300, x)
    assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.sweeps == k
    assert wait_ticks(s) == resident   # no wait ran out
    s.close()
    return x.cpu().numpy()


# most ports of a sub-circuit: 16 and 32 (two to a wavefront, an odd number of them), 36
# and 64, 51 and 96, 75 and 96 (four blocks of 32 a side), 132 and 3-D blocks with up to
# three ports a node (unsymmetric: dense operators); random cuts of every size up to 96.
# FP32 takes the dense ones a compute unit each.
@pytest.mark.parametrize("cfg,kw,res64,res32", [
    (2, dict(dims=(12, 20), block=(4, 4)), True, True),
    (2, dict(dims=(40, 40)), True, True),
    (2, dict(dims=(36, 27), block=(9, 9)), True, True),
    (1, dict(dims=(33, 64)), True, True),
    (2, dict(dims=(51, 34), block=(17, 17)), True, True),
    (2, dict(dims=(72, 72), block=(24, 24)), True, True),
    (2, dict(dims=(75, 60), block=(25, 25)), True, True),
    (2, dict(dims=(96, 96), block=(32, 32)), True, True),
    (2, dict(dims=(99, 99), block=(33, 33)), True, True),
    (3, dict(dims=(9, 10, 12), block=(3, 3, 3)), True, True),
    (3, dict(dims=(12, 12, 13), block=(4, 4, 4)), True, True),
    (4, dict(dims=(100, 90)), True, True),
])
@pytest.mark.parametrize("prec", ["fp64", "fp32_refine"])
def test_iterates(torch, cfg, kw, res64, res32, prec):
    w = workloads.make(cfg, nrhs=1, **kw)
    n_s = int(np.bincount(w.part).max())
    resident = res64 if prec == "fp64" else res32
    for k in (2, 7):
        bound = 1e-11 if prec == "fp64" else 5.5 * math.sqrt(k) * 2.0 ** -24 * math.sqrt((2 + n_s) / 3) * 8
        extra = dict() if prec == "fp64" else dict(precision=prec, max_outer=1)
        for adjoint in (False, True):
            ref = reference(w.A.T.tocsr() if adjoint else w.A, w, k)
            x = iterate(torch, w, k, resident, adjoint, **extra)
            err = np.abs(x - ref).max()
            assert err <= bound * np.abs(ref).max(), (k, adjoint, err)


@pytest.mark.parametrize("cfg,kw,opts", [
    (1, dict(), dict()),
    (1, dict(), dict(check_every=1, adaptive_checks=False)),
    (4, dict(dims=(150, 130), nrhs=1), dict(check_every=3)),
    (2, dict(dims=(200, 120)), dict(max_sweeps=100)),
    (2, dict(dims=(64, 64)), dict(check_every=1, adaptive_checks=False)),   # over 500 checks
    (5, dict(dims=(64, 64)), dict(precision="fp32_refine")),
    (2, dict(dims=(71, 64)), dict(precision="fp32_refine")),
    (5, dict(dims=(130, 117), block=(11, 13)), dict(precision="fp32_refine")),
])
def test_same_sweeps_checks_and_history_as_a_launch_per_sweep(torch, cfg, kw, opts):
    w = workloads.make(cfg, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    got = []
    for timing in (0, 1):
        s = vtm().Solver(w.A, w.part, w.Z, timing=timing, **opts)
        assert wait_ticks(s)
        x = torch.empty_like(b)
        reports = []
        for _ in range(2):
            try:
                reports.append(s.solve(b, w.tol, x)[1])
            except vtm().VTMError as e:
                assert e.name == "VTM_E_MAXITER" and "max_sweeps" in opts
                reports.append(e.report)
        assert wait_ticks(s)
        got.append((x.cpu().numpy(), reports[1]))
        s.close()
    (x0, r0), (x1, r1) = got
    assert (r0.sweeps, r0.outer, r0.checks) == (r1.sweeps, r1.outer, r1.checks)
    assert np.array_equal(r0.history_sweeps, r1.history_sweeps)
    if "precision" not in opts:
        assert np.abs(x0 - x1).max() <= 1e-11 * np.abs(x1).max()
    else:  # FP32 sweeps round alike in both
        assert np.array_equal(x0, x1)


def test_zero_right_hand_side_divergence_and_waves(torch):
    w = workloads.make(2, dims=(48, 40))
    s = vtm().Solver(w.A, w.part, w.Z, divergence=1e-30)
    x, rep = s.solve(torch.zeros((1, w.n), dtype=torch.float64, device="cuda"), 1e-8)
    assert rep.sweeps == 0 and not x.any()
    b = torch.as_tensor(w.b, device="cuda")
    with pytest.raises(vtm().VTMError) as ei:
        s.solve(b, 1e-8)
    assert ei.value.name == "VTM_E_DIVERGED" and ei.value.report.sweeps == 8
    bad = b.clone()
    bad[0, 5] = float("nan")
    with pytest.raises(vtm().VTMError) as ei:
        s.solve(bad, 1e-8)
    assert ei.value.name == "VTM_E_DIVERGED"
    assert wait_ticks(s)
    # the waves left are those of the last sweep: resumed, the solve is done at once
    s2 = vtm().Solver(w.A, w.part, w.Z)
    x2, rep2 = s2.solve(b, 1e-10)
    s2.set_waves(s2.get_waves())
    x3, rep3 = s2.solve(b, 1e-9)
    assert rep3.sweeps <= 8 and np.abs((x3 - x2).cpu().numpy()).max() <= 1e-8 * np.abs(x2.cpu().numpy()).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32_refine"])
def test_a_wait_that_runs_out_falls_back(torch, prec):
    """Every wait bounded to one try: the run ends without a result, and the solve is
    done again with a launch per sweep, now and later."""
    w = workloads.make(1)
    b = torch.as_tensor(w.b, device="cuda")
    s = vtm().Solver(w.A, w.part, w.Z, precision=prec)
    ref, r0 = s.solve(b, w.tol)
    assert wait_ticks(s, 0)
    for _ in range(2):
        x, rep = s.solve(b, w.tol)
        assert not wait_ticks(s, 0)
        assert (rep.sweeps, rep.outer, rep.checks) == (r0.sweeps, r0.outer, r0.checks)
        assert np.abs((x - ref).cpu().numpy()).max() <= 1e-9 * np.abs(ref.cpu().numpy()).max()


def test_threads_and_streams(torch):
    """Handles on four streams, solved from four host threads at once."""
    ws = [workloads.make(1, seed=k) for k in range(4)]
    streams = [torch.cuda.Stream() for _ in ws]
    bs = [torch.as_tensor(w.b, device="cuda") for w in ws]
    torch.cuda.synchronize()
    ss = [vtm().Solver(w.A, w.part, w.Z, stream=st) for w, st in zip(ws, streams)]
    want = [s.solve(b, w.tol)[0].clone() for s, b, w in zip(ss, bs, ws)]
    torch.cuda.synchronize()
    got = [None] * 4

    def work(k):
        with torch.cuda.stream(streams[k]):
            for _ in range(5):
                got[k] = ss[k].solve(bs[k], ws[k].tol)[0]

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    torch.cuda.synchronize()
    for k in range(4):
        assert torch.equal(got[k], want[k]) and wait_ticks(ss[k])
