"""Circuit.solver with conductances that change while a handle takes them, from several
streams, of other types and on other devices: the handle always holds those asked for."""
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


@pytest.fixture
def setup(torch):
    """A circuit, its conductances on the device, and a list that grows by each refresh;
    `after` of the list's attribute runs at a refresh's end."""
    from paper_0910_0663_amd import Circuit
    w = workloads.make(1, dims=(40, 33), block=(8, 8))
    c = Circuit(w.n, w.edges, w.ground, w.part, w.Z, tol=1e-10, precision="fp64")
    g = torch.as_tensor(w.g, device="cuda").clone()
    s = c.solver(g)
    seen, original, hook = [], s.refresh, []

    def refresh(*a, **k):
        original(*a, **k)
        seen.append(1)
        if hook:
            hook.pop()()

    s.refresh = refresh
    return c, g, seen, hook


def test_conductances_that_change_during_a_refresh(torch, setup):
    c, g, seen, hook = setup
    g.mul_(1.5)
    hook.append(lambda: g.mul_(2.0))      # an optimizer's step beside the refresh
    c.solver(g)
    n = len(seen)
    c.solver(g)                           # the handle holds the values before that step
    assert len(seen) == n + 1
    c.solver(g)
    assert len(seen) == n + 1


def test_two_streams(torch, setup):
    c, g, seen, hook = setup
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    first, second = g * 1.5, g * 3.0
    torch.cuda.synchronize()
    with torch.cuda.stream(one):
        c.solver(first)
        hook.append(lambda: torch.cuda._sleep(500_000_000))   # what follows on this stream comes late
        c.solver(second)
    with torch.cuda.stream(two):
        n = len(seen)
        c.solver(first)
        assert len(seen) == n + 1
    torch.cuda.synchronize()


def test_types_and_devices(torch, setup):
    c, g, seen, hook = setup
    with pytest.warns(UserWarning):
        c.solver(g.to(torch.complex128))  # the real part, as a conversion to FP64 takes it
    c.solver(g.cpu())
    assert not seen                       # the same values
    c.solver(g.to(torch.bfloat16))
    assert len(seen) == 1
    c.solver(g.to(torch.bfloat16).double().cpu())
    assert len(seen) == 1
    c.solver(g.cpu())
    c.solver(g)
    assert len(seen) == 2
