"""Port-node sweeps of dense operators, one launch per sweep, on every route that the
operators' size and the number of sub-circuits choose: the iterates of sweeps over the
full inverses (local_form "full", which other tests hold to the oracle's).

Tolerance: both forms round dot products of at most n_s = 1,000 terms, n_s u sqrt-wise
5.5 sqrt(k) u sqrt((2 + n_s) / 3) 8 of max |x| over k contracting sweeps, u = 2^-53 or
2^-24; twice that between two rounded results.
"""
import math

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
K = 5


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


# sub-circuits, port nodes of the largest, MB of operators.  FP64: nearly as many as the
# compute units (a workgroup each) and too few for that (rows over workgroups); between one
# and two a unit, within the cache, above it (alternating) and above twice it (non-temporal);
# rows over workgroups, alternating and non-temporal.  FP32: the same sizes of operators.
@pytest.mark.parametrize("prec,dims,block,S,mb", [
    ("fp64", (54, 54, 45), 9, 180, (100, 256)), ("fp64", (45, 54, 45), 9, 150, (0, 256)),
    ("fp64", (40, 48, 80), 8, 300, (0, 256)), ("fp64", (54, 54, 90), 9, 360, (256, 512)), ("fp64", (56, 56, 80), 8, 490, (256, 512)),
    ("fp64", (60, 60, 100), 10, 360, (512, 2048)), ("fp64", (64, 64, 64), 8, 512, (256, 512)),
    ("fp64", (80, 80, 80), 8, 1000, (512, 2048)),
    ("fp32_refine", (48, 48, 40), 8, 180, (0, 256)), ("fp32_refine", (80, 80, 80), 8, 1000, (256, 512)),
    ("fp32_refine", (100, 96, 98), 8, 2028, (512, 2048)),
])
def test_iterates(torch, prec, dims, block, S, mb):
    import paper_0910_0663_amd as vtm
    w = workloads.make(3, nrhs=1, dims=dims, block=(block,) * 3)
    b = torch.as_tensor(w.b, device="cuda")
    extra = dict() if prec == "fp64" else dict(precision=prec, max_outer=1)
    got = []
    for form in ("port", "full"):
        s = vtm.Solver(w.A, w.part, w.Z, check_every=K, max_sweeps=K, adaptive_checks=False, timing=1,
                       local_form=form, **extra)
        assert s.n_sub == S
        if form == "port":
            assert mb[0] < s.port_operator_bytes / 2 ** 20 <= mb[1]
        x = torch.empty_like(b)
        with pytest.raises(vtm.VTMError) as ei:
            s.solve(b, 1e-300, x)
        assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.sweeps == K
        got.append(x.cpu().numpy())
        s.close()
    u = 2.0 ** -53 if prec == "fp64" else 2.0 ** -24
    bound = 2 * 5.5 * math.sqrt(K) * u * math.sqrt((2 + block ** 3) / 3) * 8
    err = np.abs(got[0] - got[1]).max()
    assert err <= bound * np.abs(got[1]).max(), err
