"""Check intervals captured as graphs, on sweeps that are not resident: one column of
circuits too large for it and several columns, eager against replayed, bit for bit.

Each solve replays its graphs many times, with the host's own eager work and
synchronisations in between.
"""
import ctypes as C

import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


# one column: packed operators two to a wavefront (more sub-circuits than the chip holds) and
# one over eight wavefronts; dense ones of more than 320 port nodes, in both directions.
# Several columns: tiles in up to 64 KiB of LDS and above (16 x 16 x 16, 12 columns), on the
# transposed ones for the adjoint, FP32, and the dense port operator
@pytest.mark.parametrize("cfg,kw,prec,nrhs,form", [
    (2, dict(dims=(800, 704), block=(8, 8)), "fp64", 1, "port"),
    (2, dict(dims=(800, 704), block=(8, 8)), "fp32_refine", 1, "port"),
    (2, dict(dims=(640, 656), block=(16, 16)), "fp64", 1, "port"),
    (2, dict(dims=(640, 656), block=(16, 16)), "fp32_refine", 1, "port"),
    (3, dict(dims=(27, 27, 18), block=(9, 9, 9)), "fp64", 1, "port"),
    (3, dict(dims=(27, 27, 18), block=(9, 9, 9)), "fp32_refine", 1, "port"),
    (2, dict(dims=(64, 60)), "fp64", 3, "port"), (2, dict(dims=(64, 60)), "fp32_refine", 7, "port"),
    (3, dict(dims=(16, 16, 16)), "fp64", 12, "port"), (3, dict(dims=(16, 16, 12)), "fp32_refine", 5, "port"),
    (2, dict(dims=(64, 60)), "fp64", 4, "port_dense"), (2, dict(dims=(64, 60)), "fp64", 1, "port_dense"),
])
def test_replay_matches_eager_bitwise(torch, cfg, kw, prec, nrhs, form):
    import paper_0910_0663_amd as vtm
    is_resident = vtm.lib().vtm_testing_wait_ticks
    is_resident.argtypes, is_resident.restype = [C.c_void_p, C.c_uint64], C.c_int
    w = workloads.make(cfg, nrhs=nrhs, **kw)
    b = torch.as_tensor(w.b, device="cuda")
    common = dict(precision=prec, nrhs_max=nrhs, check_every=4, adaptive_checks=False, local_form=form)
    graph = vtm.Solver(w.A, w.part, w.Z, use_graph=True, **common)
    eager = vtm.Solver(w.A, w.part, w.Z, **common)
    assert nrhs > 1 or not is_resident(graph._h, 400_000_000)
    for adjoint in (False, True):
        got = []
        for s in (graph, graph, graph, eager):
            x, end = torch.empty_like(b), "VTM_OK"
            try:
                rep = (s.solve_adjoint if adjoint else s.solve)(b, 1e-8, x)[1]
            except vtm.VTMError as e:   # checks every 4 sweeps end FP32 inner solves early, as stalled
                end, rep = e.name, e.report
            torch.cuda.synchronize()
            assert end == "VTM_OK" or (prec, end) == ("fp32_refine", "VTM_E_MAXITER")
            got.append((x, (end, rep.sweeps, rep.outer, rep.checks)))
        for x, r in got[:3]:
            assert r == got[3][1] and torch.equal(x, got[3][0])
    graph.close()
    eager.close()
