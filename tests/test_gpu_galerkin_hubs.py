"""AMG hierarchies with hub rows: member lists and coarse rows of more than 1,024.

One matching round leaves most rows to join the pairs it found, so strongly
heterogeneous fields grow hubs that thousands of rows belong to.  Lists and
products with more than 1,024 members or terms in a row are sorted instead of
compared entry by entry, and the levels of such lists are not fused in the
cycle.  Checked: the first level's aggregates and pattern against the oracle's;
every coarse matrix against P^T A P (t terms, grouped in another way where a
level takes several passes, are off by at most t eps of the sum of their
magnitudes); a cycle against NumPy on the exported levels in the bound of the
cycle test (four times eps times the longest row times the sweeps times the
coarsest matrix's condition).  Two cases pass the rule for terms only.
"""
import numpy as np
import pytest

import workloads
from test_gpu_amg_levels import _cycle

pytestmark = pytest.mark.gpu

# nx, ny, nz, sigma, passes, rounds, theta, has hubs
CASES = [(60, 60, 20, 2.0, 4, 1, 0.25, True), (60, 60, 20, 6.0, 1, 1, 0.0, True),
         (40, 30, 9, 6.0, 2, 1, 0.25, False), (101, 97, 23, 4.0, 2, 1, 0.25, True),
         (101, 97, 23, 6.0, 3, 4, 0.25, False)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_hierarchy_and_cycle(case):
    import scipy.sparse as sp
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_1701_06254_amd import r2p
    nx, ny, nz, sigma, passes, rounds, theta, hubs = case
    w = workloads.make_gaussian(nx, ny, nz, seed=1, sigma=sigma)
    mo, m = oracle.Model(w), r2p.Model(w)
    xh = workloads.random_state(w, np.random.default_rng(nx), p_spread=5.0)
    x = torch.as_tensor(xh, device="cuda")
    J = r2p.Jacobian(m)
    J.assemble(x, m.initial_state(), 2.0)
    kw = dict(px=1, py=1, max_coarse=200, agg_passes=passes, match_rounds=rounds, theta=theta,
              max_levels=12, kcycle=0, amg_cycles=1)
    P = r2p.Cpr().setup(J, r2p.cpr_opts(**kw))
    L = P.amg_levels()
    Jo, F = mo.jacobian(xh, mo.initial_state(), 2.0)
    Ad, _ = oracle.decouple(Jo, -F, mo.n, oracle.DEC_QI)
    Lo = oracle.Amg(oracle.extract_pressure(Ad, mo.n), theta, 200, 12, rounds, passes)
    assert np.array_equal(L[0]["agg"], Lo.level(0)["agg"])
    assert np.array_equal(L[1]["rp"], Lo.level(1)["A"].rp)
    assert np.array_equal(L[1]["col"], Lo.level(1)["A"].col)
    for l in L:
        l["A"] = sp.csr_matrix((l["val"], l["col"], l["rp"]), shape=(l["n"], l["n"]))
    members = terms = 0
    for f, c in zip(L, L[1:]):
        R = sp.csr_matrix((np.ones(f["n"]), (f["agg"], np.arange(f["n"]))), shape=(c["n"], f["n"]))
        ref, mag = (R @ f["A"] @ R.T).tocsr(), (R @ abs(f["A"]) @ R.T).tocsr()
        cnt = (R @ sp.csr_matrix((np.ones_like(f["val"]), f["col"], f["rp"]), shape=f["A"].shape) @ R.T).tocsr()
        for M in (ref, mag, cnt):
            M.sort_indices()
        assert np.array_equal(cnt.indptr, c["rp"]) and np.array_equal(cnt.indices, c["col"])
        bound = cnt.multiply(mag) * np.finfo(float).eps
        assert (abs(c["A"] - ref) - bound).max() <= 0.0
        members = max(members, np.bincount(f["agg"]).max())
        terms = max(terms, np.asarray(cnt.sum(axis=1)).max())
    assert terms > 1024 and (members > 1024) == hubs
    f = np.random.default_rng(2).standard_normal(m.n)
    got = P.amg_vcycle(torch.as_tensor(f, device="cuda")).cpu().numpy()
    ref = _cycle(L, 0, f, 0)
    longest = max(np.diff(l["rp"]).max() for l in L)
    tol = (4 * np.finfo(float).eps * longest * (2 * len(L) + 1)
           * np.linalg.cond(L[-1]["A"].toarray()))
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
