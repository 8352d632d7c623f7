"""Every coarse AMG matrix against P^T A P of the level above.

Two aggregation passes make a level, so the two sides group the same terms
differently: t terms are off by at most t eps of the sum of their magnitudes.
The stored pattern is the product's, columns ascending.  The sizes run from
single rows to levels whose coarse rows have more than 64 terms and aggregates
of more than 16 members, which take a path of their own.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("passes", [1, 2, 3])
@pytest.mark.parametrize("nx,ny,nz", [(2, 1, 1), (17, 1, 1), (16, 16, 1), (29, 23, 7), (101, 97, 23)])
def test_levels_are_galerkin_products(nx, ny, nz, passes):
    import scipy.sparse as sp
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    w = workloads.make_gaussian(nx, ny, nz, seed=1) if nx == 101 else workloads.make_tiny(nx, ny, nz)
    m = r2p.Model(w)
    x = torch.as_tensor(workloads.random_state(w, np.random.default_rng(nx), p_spread=5.0), device="cuda")
    J = r2p.Jacobian(m)
    J.assemble(x, m.initial_state(), 2.0)
    P = r2p.Cpr().setup(J, r2p.cpr_opts(px=1, py=1, max_coarse=1, agg_passes=passes, max_levels=12))
    L = P.amg_levels()
    for l in L:
        l["A"] = sp.csr_matrix((l["val"], l["col"], l["rp"]), shape=(l["n"], l["n"]))
    terms = 0
    for f, c in zip(L, L[1:]):
        R = sp.csr_matrix((np.ones(f["n"]), (f["agg"], np.arange(f["n"]))), shape=(c["n"], f["n"]))
        ref = (R @ f["A"] @ R.T).tocsr()
        cnt = (R @ sp.csr_matrix((np.ones_like(f["val"]), f["col"], f["rp"]), shape=f["A"].shape) @ R.T).tocsr()
        mag = (R @ abs(f["A"]) @ R.T).tocsr()
        for M in (ref, cnt, mag):
            M.sort_indices()
        assert np.array_equal(cnt.indptr, c["rp"]) and np.array_equal(cnt.indices, c["col"])
        terms = max(terms, np.asarray(cnt.sum(axis=1)).max())
        d = abs(c["A"] - ref)
        bound = cnt.multiply(mag) * np.finfo(float).eps
        assert (d - bound).max() <= 0.0
    if nx == 101:
        assert terms > 64 and max(np.bincount(l["agg"]).max() for l in L[:-1]) > 16
