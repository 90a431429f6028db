"""Device memory that does not suffice for everything a handle would like to keep: second
copies of operators for several right-hand sides, transposed ones for an adjoint and the
exchange words of resident runs are given up, never the handle.

The library's own bound on the calling thread's memory (vtm_testing_memory) stands for a
device that is full.  Results keep the relative residual asked for, 1e-8, in every case.
"""
import ctypes as C

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
PLENTY = 1 << 40


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


@pytest.fixture
def bound():
    import paper_0910_0663_amd as vtm
    f = vtm.lib().vtm_testing_memory
    f.argtypes, f.restype = [C.c_int64], C.c_int64
    yield f
    f(-1)


def solve_both(torch, s, w, nrhs):
    b = torch.as_tensor(w.b, device="cuda")
    A = w.A.tocsr()
    for solve, M in ((s.solve, A), (s.solve_adjoint, A.T.tocsr())):
        x = solve(b, 1e-8)[0].cpu().numpy()
        for r in range(nrhs):
            res = w.b[r] - M @ x[r]
            assert np.linalg.norm(res) <= 1.01e-8 * np.linalg.norm(w.b[r])


# packed operators and dense ones (transposes, too) with tiles for several columns; batched
# tiles with transposed port operators; the dense port operator; one column, resident.  The
# last value: whether less is enough than all of it takes (sub-circuits of 512 nodes need
# more for their temporary inverses than the copies take afterwards)
CASES = [
    ("fp64", 2, dict(dims=(64, 60)), 6, "port", True), ("fp32_refine", 2, dict(dims=(64, 60)), 4, "port", True),
    ("fp64", 3, dict(dims=(16, 16, 16)), 3, "port", False), ("fp32_refine", 3, dict(dims=(16, 16, 12)), 3, "port", False),
    ("fp64", 3, dict(dims=(16, 16, 12)), 16, "port", True), ("fp64", 2, dict(dims=(64, 60)), 5, "port_dense", True),
    ("fp64", 2, dict(dims=(64, 60)), 1, "port", True), ("fp64", 2, dict(dims=(64, 60)), 16, "port", False),
]


@pytest.mark.parametrize("prec,cfg,kw,nrhs,form,optional", CASES)
def test_setup_takes_what_it_must_first(torch, bound, prec, cfg, kw, nrhs, form, optional):
    """What is enough once is enough with more; with less than everything, but enough,
    the handle works."""
    import paper_0910_0663_amd as vtm
    w = workloads.make(cfg, nrhs=nrhs, **kw)

    def make(limit):
        bound(limit)
        try:
            return vtm.Solver(w.A, w.part, w.Z, precision=prec, nrhs_max=nrhs, local_form=form)
        finally:
            make.low = bound(-1)

    make(PLENTY).close()
    whole = PLENTY - make.low
    enough = []
    for limit in np.linspace(whole / 2, whole, 49, dtype=np.int64):
        try:
            s = make(int(limit))
        except vtm.VTMError as e:
            assert e.name == "VTM_E_OOM"
            assert not enough, f"{enough[0]} bytes were enough, {limit} are not"
            continue
        if not enough or limit == whole:
            solve_both(torch, s, w, nrhs)
        enough.append(int(limit))
        s.close()
    assert enough and (enough[0] < whole) == optional


@pytest.mark.parametrize("prec,cfg,kw,nrhs", [
    ("fp64", 1, dict(dims=(70, 66), block=(33, 33)), 6), ("fp32_refine", 1, dict(dims=(70, 66), block=(33, 33)), 4),
    ("fp64", 3, dict(dims=(16, 16, 16)), 3), ("fp64", 3, dict(dims=(16, 16, 12)), 16),
])
def test_refresh_gives_up_what_it_can(torch, bound, prec, cfg, kw, nrhs):
    """A refresh that lacks one byte for its temporary inverses finds them in the copies
    that the handle can do without."""
    import paper_0910_0663_amd as vtm
    w = workloads.make(cfg, nrhs=nrhs, **kw)
    s = vtm.Solver(w.A, w.part, w.Z, precision=prec, nrhs_max=nrhs)
    bound(PLENTY)
    s.refresh(w.A)
    need = PLENTY - bound(-1)
    assert need > 0
    solve_both(torch, s, w, nrhs)
    bound(need - 1)
    s.refresh(w.A)
    bound(-1)
    solve_both(torch, s, w, nrhs)
    s.close()
