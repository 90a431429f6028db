"""Control of resident runs: long intervals between checks, more checks than a launch
reports, and the exchange words' tags at the end of their range.

timing = 1 takes a launch per sweep.  FP64 iterates 1e-11 of max |x| (dot products of at most
n_s = 512 terms, n_s 2^-53 = 6e-14 each, over contracting sweeps); a check's relative
residual ||A dx|| / ||b|| then differs by at most 2 max |A_ii| 1e-11 max |x| sqrt(n) / ||b||
(rows of A sum to at most twice their diagonal), and by the rounding of its own sums, 1e-12 of
it.  FP32 sweeps round alike in both.
"""
import ctypes as C

import numpy as np
import pytest

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


def epoch(s, value):
    f = vtm().lib().vtm_testing_epoch
    f.argtypes, f.restype = [C.c_void_p, C.c_uint32], C.c_uint32
    return f(s._h, value)


def resident(s, ticks=400_000_000):
    f = vtm().lib().vtm_testing_wait_ticks
    f.argtypes, f.restype = [C.c_void_p, C.c_uint64], C.c_int
    return bool(f(s._h, ticks))


# an interval of 8,192 or 16,384 sweeps takes 13 to 70 ms: several times a bound of 2 ms, which
# no single sweep takes
@pytest.mark.parametrize("cfg,kw,prec,every", [
    (1, dict(), "fp64", 16384), (1, dict(), "fp32_refine", 16384),
    (3, dict(dims=(24, 24, 24), block=(8, 8, 8)), "fp64", 8192),
    (3, dict(dims=(24, 24, 24), block=(8, 8, 8)), "fp32_refine", 8192),
])
def test_an_interval_longer_than_the_bound_of_a_wait(torch, cfg, kw, prec, every):
    w = workloads.make(cfg, nrhs=1, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    s = vtm().Solver(w.A, w.part, w.Z, precision=prec, check_every=every, adaptive_checks=False)
    s.solve(b, 1e-8)
    assert resident(s, 200_000)
    x, rep = s.solve(b, 1e-8)
    assert resident(s)
    assert rep.sweeps % every == 0 and rep.relres_max <= 1e-8
    s.close()


# 1,500 checks of one sweep each: a launch reports 1,024 of them
@pytest.mark.parametrize("cfg,kw", [
    (1, dict()), (2, dict(dims=(40, 44))), (3, dict(dims=(16, 16, 16), block=(8, 8, 8))),
])
def test_more_checks_than_a_launch_reports(torch, cfg, kw):
    w = workloads.make(cfg, nrhs=1, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    got = []
    for timing in (0, 1):
        s = vtm().Solver(w.A, w.part, w.Z, timing=timing, check_every=1, adaptive_checks=False, max_sweeps=1500)
        x = torch.empty_like(b)
        with pytest.raises(vtm().VTMError) as ei:
            s.solve(b, 1e-300, x)
        assert ei.value.name == "VTM_E_MAXITER" and resident(s)
        got.append((x.cpu().numpy(), ei.value.report))
        s.close()
    (x0, r0), (x1, r1) = got
    assert r0.sweeps == r1.sweeps == 1500 and r0.checks == r1.checks >= 1500
    assert np.array_equal(r0.history_sweeps, r1.history_sweeps)
    assert np.abs(x0 - x1).max() <= 1e-11 * np.abs(x1).max()
    bound = 2 * w.A.diagonal().max() * 1e-11 * np.abs(x1).max() * np.sqrt(w.n) / np.linalg.norm(w.b)
    assert (np.abs(r0.history - r1.history) <= bound + 1e-12 * r1.history).all()


@pytest.mark.parametrize("cfg,kw,prec", [
    (1, dict(), "fp64"), (4, dict(dims=(150, 130)), "fp64"), (1, dict(), "fp32_refine"), (5, dict(dims=(64, 64)), "fp32_refine"),
    (3, dict(dims=(16, 16, 16), block=(8, 8, 8)), "fp64"), (3, dict(dims=(16, 16, 16), block=(8, 8, 8)), "fp32_refine"),
])
def test_history_values(torch, cfg, kw, prec):
    w = workloads.make(cfg, nrhs=1, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    got = []
    for timing in (0, 1):
        s = vtm().Solver(w.A, w.part, w.Z, timing=timing, precision=prec)
        x, rep = s.solve(b, w.tol)
        assert resident(s)
        got.append((x.cpu().numpy(), rep))
        s.close()
    (x0, r0), (x1, r1) = got
    assert np.array_equal(r0.history_sweeps, r1.history_sweeps)
    if prec == "fp64":
        bound = 2 * w.A.diagonal().max() * 1e-11 * np.abs(x1).max() * np.sqrt(w.n) / np.linalg.norm(w.b)
        assert (np.abs(r0.history - r1.history) <= bound + 1e-12 * r1.history).all()
    else:
        assert np.array_equal(x0, x1) and np.array_equal(r0.history, r1.history)


@pytest.mark.parametrize("cfg,kw,prec", [
    (1, dict(), "fp64"), (1, dict(), "fp32_refine"),
    (2, dict(dims=(368, 240)), "fp64"),                                    # sixteen sub-circuits a workgroup
    (3, dict(dims=(16, 16, 16), block=(8, 8, 8)), "fp64"), (3, dict(dims=(16, 16, 16), block=(8, 8, 8)), "fp32_refine"),
])
def test_the_words_are_cleared_before_their_tags_run_out(torch, cfg, kw, prec):
    w = workloads.make(cfg, nrhs=1, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    s = vtm().Solver(w.A, w.part, w.Z, precision=prec)
    x, rep = s.solve(b, w.tol)
    last = 2 ** 32 - 1 - 2 ** 28
    assert 0 < epoch(s, last) <= rep.sweeps + 1
    for k in range(4):                    # up to the last tag a run may start from, past it, then from 0 again
        y, r = s.solve(b, w.tol)
        assert torch.equal(x, y) and (r.sweeps, r.checks) == (rep.sweeps, rep.checks) and resident(s)
    assert epoch(s, 0) < 5 * rep.sweeps
    s.close()
