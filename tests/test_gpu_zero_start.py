"""The start from x = 0, whose residual is b without a pass over A, and the solves that
end there: a zero right-hand side, no outer step allowed, a source that is not a number.
Each after a solve that left another x in the handle's buffers; exact values throughout."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


# resident and a launch per sweep (timing), one and several columns, the batched tiles,
# wires and vertices
@pytest.mark.parametrize("precision,nrhs,opts", [
    ("fp64", 1, {}), ("fp64", 1, dict(timing=1)), ("fp64", 1, dict(check_every=1, adaptive_checks=False)),
    ("fp64", 3, {}), ("fp64", 16, {}), ("fp32_refine", 1, {}), ("fp32_refine", 1, dict(timing=1)),
    ("fp32_refine", 3, {}), ("bf16_refine", 64, {}),
])
def test_zero_right_hand_side(torch, precision, nrhs, opts):
    import paper_0910_0663_amd as vtm
    w = workloads.make(2, nrhs=1, dims=(64, 48))
    rng = np.random.default_rng(3)
    b = torch.as_tensor(rng.standard_normal((nrhs, w.n)), device="cuda")
    s = vtm.Solver(w.A, w.part, w.Z, precision=precision, nrhs_max=nrhs, **opts)
    want, r0 = s.solve(b, w.tol)
    assert r0.history[0] == 1.0 and r0.history_sweeps[0] == 0
    x = torch.full_like(b, 7.0)
    _, rep = s.solve(torch.zeros_like(b), w.tol, x)
    assert not x.any() and (rep.sweeps, rep.checks, rep.outer) == (0, 1, 0)
    assert rep.relres_max == 0.0 and list(rep.history) == [0.0]
    if precision == "fp64":
        assert not s.get_waves(nrhs).any()
    again, r1 = s.solve(b, w.tol)
    assert torch.equal(again, want) and (r1.sweeps, r1.checks) == (r0.sweeps, r0.checks)
    # a tolerance that x = 0 meets
    _, rep = s.solve(b, 1.0, x)
    assert not x.any() and rep.sweeps == 0


@pytest.mark.parametrize("precision", ["fp32_refine", "bf16_refine"])
def test_no_outer_step(torch, precision):
    import paper_0910_0663_amd as vtm
    w = workloads.make(2, nrhs=1, dims=(64, 48))
    nrhs = 16 if precision == "bf16_refine" else 1
    b = torch.as_tensor(np.repeat(w.b, nrhs, 0), device="cuda")
    s = vtm.Solver(w.A, w.part, w.Z, precision=precision, nrhs_max=nrhs, max_outer=1)
    x = torch.full_like(b, 7.0)
    with pytest.raises(vtm.VTMError) as ei:
        s.solve(b, 1e-300, x)
    assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.outer == 1 and x.any()
    bad = b.clone()
    bad[0, 5] = float("nan")
    with pytest.raises(vtm.VTMError) as ei:
        s.solve(bad, 1e-8, x)
    assert ei.value.name == "VTM_E_DIVERGED" and ei.value.report.sweeps == 0 and not x.any()
    s.close()
    s = vtm.Solver(w.A, w.part, w.Z, precision=precision, nrhs_max=nrhs, max_outer=0)
    x.fill_(7.0)
    with pytest.raises(vtm.VTMError) as ei:
        s.solve(b, 1e-8, x)
    assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.sweeps == 0 and not x.any()
