"""Circuit.solver notices every change of the conductances, however they come, and
only a change: the handle's values equal those of a fresh one, bit for bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


def make(w):
    from paper_0910_0663_amd import Circuit
    return Circuit(w.n, w.edges, w.ground, w.part, w.Z, tol=1e-10, precision="fp64")


@pytest.mark.parametrize("where", ["cuda", "cpu"])
def test_changes_of_the_conductances(torch, where):
    w = workloads.make(1, dims=(40, 33), block=(8, 8))
    b = torch.as_tensor(w.b, device="cuda")
    g = torch.as_tensor(w.g, device=where).clone()
    c = make(w)
    refreshed = []

    def check(gt, changed):
        s = c.solver(gt)
        if not refreshed:
            original = s.refresh
            s.refresh = lambda *a, **k: (refreshed.append(1), original(*a, **k))[1]
        n = len(refreshed)
        s = c.solver(gt)                      # the same values again: nothing to do
        assert len(refreshed) == n
        fresh = make(w).solver(gt.detach().clone())
        assert torch.equal(s.solve(b, 1e-10)[0], fresh.solve(b, 1e-10)[0])
        return s

    s0 = check(g, True)
    refreshed.append(0)                       # from here on counted
    for k, change in enumerate((lambda: g.__setitem__(7, g[7] * 1.5),                 # in place
                                lambda: g.mul_(1.01),
                                lambda: g.__setitem__(-1, g[-1] * (1 + 2 ** -50)))):  # one value, its last bits
        change()
        n = len(refreshed)
        c.solver(g)
        assert len(refreshed) == n + 1
        assert check(g, False) is s0
    # another tensor of the same values, strided; another type; back
    wide = torch.empty((g.numel(), 2), dtype=g.dtype, device=where)
    wide[:, 0] = g
    n = len(refreshed)
    assert c.solver(wide[:, 0]) is s0 and len(refreshed) == n
    c.solver(g.to(torch.float32))
    assert len(refreshed) == n + 1
    check(g.to(torch.float32), False)
    # a refused refresh leaves nothing to be taken for done
    bad = g.clone()
    bad[3] = float("nan")
    for _ in range(2):
        with pytest.raises(Exception):
            c.solver(bad)
    check(g, True)
