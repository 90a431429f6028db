"""Port-to-port sweeps of several right-hand sides on column-group handles: the
port-node tiles on the matrix cores and the dense port operator, against the
oracle's iterates.

x^k follows a first full sweep, k - 2 port-to-port sweeps and a last full sweep
(check_every = k).  FP64 tolerance: each sweep rounds dot products of at most
n_s <= 512 terms (n_s 2^-53 ~ 6e-14) and the iteration contracts (rho <= 0.99), so
the difference stays below 6e-12 of max |x|; 1e-11 is used.  FP32: n_s terms
with two roundings each and their partial sums, 5.5 sqrt(k) u sqrt((2 + n_s) / 3) 8
of max |x| with u = 2^-24 (5.5 standard deviations; sum |K^-1_ij rhs_j| <= 8 max |x|
on these circuits).
"""
import math

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

K = 6


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a HIP device"
    return T


def vtm():
    import paper_0910_0663_amd as v
    return v


def reference(torn, b, k=K):
    sw = oracle.Sweeper(torn)
    a = np.zeros((2, torn.n_lines, b.shape[0]))
    for _ in range(k):
        u, a = sw.sweep(torn.src @ b.T, a)
    return (torn.out @ u).T


def iterate(torch, make, b, adjoint=False, refine=False):
    s = make(check_every=K, max_sweeps=K, adaptive_checks=False, nrhs_max=b.shape[0],
             **(dict(precision="fp32_refine", max_outer=1) if refine else {}))
    x = torch.empty(b.shape, dtype=torch.float64, device="cuda")
    bd = torch.as_tensor(np.ascontiguousarray(b), device="cuda")
    with pytest.raises(vtm().VTMError) as ei:
        (s.solve_adjoint if adjoint else s.solve)(bd, 1e-300, x)
    assert ei.value.name == "VTM_E_MAXITER" and ei.value.report.sweeps == K
    s.close()
    return x.cpu().numpy()


def close(x, ref, rtol):
    err, scale = np.abs(x - ref).max(), np.abs(ref).max()
    assert err <= rtol * scale, f"max err {err:.3e} vs {rtol:.2e} * {scale:.3e}"


# 8x8 blocks: 28 port nodes (two row tiles, the second ragged), 2 items a thread and,
# at 16 columns, 4; 16x16 blocks: 60 of 64 rows; random cuts up to 92 port nodes; 3-D 8^3
# blocks: 296 port nodes on 8 wavefronts, items read again; 15, 16 and 17 right-hand sides
# end a column block short, exactly and one past; 1-wide pieces and a lone node
@pytest.mark.parametrize("cfg,kw,nrhs", [
    (2, dict(dims=(40, 33)), 2),
    (2, dict(dims=(33, 40)), 7),
    (2, dict(dims=(32, 25), block=(8, 8)), 15),
    (1, dict(dims=(49, 64)), 5),
    (1, dict(dims=(49, 65)), 13),
    (4, dict(dims=(70, 61)), 6),
    (3, dict(dims=(16, 16, 16)), 3),
    (3, dict(dims=(17, 16, 9)), 12),
])
@pytest.mark.parametrize("adjoint", [False, True])
def test_fp64_iterates(torch, cfg, kw, nrhs, adjoint):
    w = workloads.make(cfg, nrhs=nrhs, **kw)
    A = w.A.T.tocsr() if adjoint else w.A
    ref = reference(oracle.tear_wires(A, w.part, w.Z), w.b)
    x = iterate(torch, lambda **o: vtm().Solver(w.A, w.part, w.Z, **o), w.b, adjoint)
    close(x, ref, 1e-11)


@pytest.mark.parametrize("cfg,kw,nrhs", [
    (2, dict(dims=(40, 33)), 3),
    (1, dict(dims=(49, 64)), 16),
    (1, dict(dims=(49, 64)), 17),
    (4, dict(dims=(70, 61)), 40),
    (3, dict(dims=(16, 16, 16)), 5),
])
def test_fp32_iterates(torch, cfg, kw, nrhs):
    w = workloads.make(cfg, nrhs=nrhs, **kw)
    n_s = int(np.bincount(w.part).max())
    x = iterate(torch, lambda **o: vtm().Solver(w.A, w.part, w.Z, **o), w.b, refine=True)
    close(x, reference(oracle.tear_wires(w.A, w.part, w.Z), w.b),
          5.5 * math.sqrt(K) * 2.0 ** -24 * math.sqrt((2 + n_s) / 3) * 8)


# the dense operator: forced (local_form 2) on 32 and 64 ports, coupled lines on few
# sub-circuits (16 to 130 ports: rows over workgroups, columns over wavefronts)
@pytest.mark.parametrize("block,nrhs", [((8, 8), 2), ((16, 16), 9)])
def test_dense_port_operator(torch, block, nrhs):
    w = workloads.make(2, dims=(48, 49), block=block, nrhs=nrhs)
    x = iterate(torch, lambda **o: vtm().Solver(w.A, w.part, w.Z, local_form="port_dense", **o), w.b)
    close(x, reference(oracle.tear_wires(w.A, w.part, w.Z), w.b), 1e-11)


@pytest.mark.parametrize("dims,width", [((8, 23), 5), ((33, 35), 8), ((65, 23), 5), ((64, 23), 5)])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 9])
def test_coupled_lines(torch, dims, width, nrhs):
    rng = np.random.default_rng(5)
    e = workloads.grid2d_edges(*dims)
    n = int(np.prod(dims))
    A = workloads.nodal_matrix(n, e, rng.uniform(0.5, 2.0, e.shape[0]), np.full(n, workloads.GROUND_S))
    b = rng.standard_normal((nrhs, n))
    label, iface, sides = workloads.separator_strips(dims, width)
    W = vtm().vertex_admittance(A, label, iface, sides, "ob")
    x = iterate(torch, lambda **o: vtm().Solver(A, label, None, iface=iface, sides=sides, W=W, **o), b)
    close(x, reference(oracle.tear_at_vertices(A, label, iface, sides, W.toarray()), b), 1e-11)
