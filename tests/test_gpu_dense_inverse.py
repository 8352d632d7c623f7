"""The coarsest AMG level's dense inverse over its range of sizes.

With one level the AMG cycle is x = A_pp^-1 f through the stored inverse.
The sizes sit at the edges of the panel width (32 columns, 16 above 1,024
rows, 8 above 2,048) and of the rows a wavefront's lanes hold (multiples of
64, 128, 256, 512, 1,024).  Bound: the explicit inverse of an LU with partial
pivoting has a forward error of at most a small multiple of n eps cond(A),
4 n eps cond_2(A) here, against a dense solve in FP64.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (1, 2, 1), (31, 1, 1), (32, 1, 1), (11, 3, 1), (63, 1, 1), (8, 8, 1), (13, 5, 1),
         (16, 8, 1), (43, 3, 1), (16, 16, 1), (257, 1, 1), (26, 18, 1), (32, 16, 1), (27, 19, 1),
         (32, 32, 1), (41, 25, 1), (32, 32, 2), (683, 3, 1), (64, 64, 1)]


@pytest.mark.parametrize("nx,ny,nz", SIZES)
def test_single_level_cycle_is_the_dense_solve(nx, ny, nz):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    n = nx * ny * nz
    w = workloads.make_tiny(nx, ny, nz)
    w["wells"] = w["wells"][:1]
    m = r2p.Model(w)
    x = m.initial_state()
    J = r2p.Jacobian(m)
    J.assemble(x, x, 5.0)
    P = r2p.Cpr().setup(J, r2p.cpr_opts(px=1, py=1, max_levels=1, max_coarse=2048))
    L = P.amg_levels()
    assert len(L) == 1 and L[0]["n"] == n
    A = np.zeros((n, n))
    rows = np.repeat(np.arange(n), np.diff(L[0]["rp"]))
    A[rows, L[0]["col"]] = L[0]["val"]
    f = np.random.default_rng(n).standard_normal(n)
    got = P.amg_vcycle(torch.as_tensor(f, device="cuda")).cpu().numpy()
    ref = np.linalg.solve(A, f)
    tol = 4 * n * np.finfo(float).eps * np.linalg.cond(A)
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("nx,ny,nz", SIZES)
def test_with_row_exchanges(nx, ny, nz):
    """At a rough state A_pp is far from diagonally dominant: the LU exchanges
    rows, also between panels, so positions and rows differ."""
    import scipy.linalg as la
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    n = nx * ny * nz
    w = workloads.make_tiny(nx, ny, nz)
    w["wells"] = w["wells"][:1]
    m = r2p.Model(w)
    x = torch.as_tensor(workloads.random_state(w, np.random.default_rng(n), p_spread=50.0), device="cuda")
    J = r2p.Jacobian(m)
    J.assemble(x, x, 5.0)
    P = r2p.Cpr().setup(J, r2p.cpr_opts(px=1, py=1, max_levels=1, max_coarse=2048))
    L = P.amg_levels()
    assert len(L) == 1 and L[0]["n"] == n
    A = np.zeros((n, n))
    rows = np.repeat(np.arange(n), np.diff(L[0]["rp"]))
    A[rows, L[0]["col"]] = L[0]["val"]
    piv, k = la.lu_factor(A)[1], np.arange(n)
    if n > 30:
        assert (piv != k).any()
    width = 32 if n <= 1024 else (16 if n <= 2048 else 8)
    if n > 2 * width:
        assert (piv // width != k // width).any()
    f = np.random.default_rng(n).standard_normal(n)
    got = P.amg_vcycle(torch.as_tensor(f, device="cuda")).cpu().numpy()
    ref = np.linalg.solve(A, f)
    tol = 4 * n * np.finfo(float).eps * np.linalg.cond(A)
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
