"""Control of resident runs: long intervals between checks, more checks than a launch
reports, and the exchange words' tags at the end of their range.

timing = 1 takes a launch per sweep.
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
