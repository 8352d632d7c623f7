"""Scans over lengths at the limits of their three forms, through what they index.

A model of n cells scans arrays of n + 1 entries in its AMG set-up: one
workgroup up to 16,384 entries, two passes up to 4,194,304, three beyond.  The row
pointers, aggregate numbers and coarse patterns of the first levels are whole
numbers: they are compared exactly with the grid's pattern and its images.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (63, 65, 1), (64, 64, 1), (129, 127, 1), (128, 128, 1),
                                      (64, 64, 4), (65, 63, 5), (2048, 2048, 1), (2047, 2049, 1)])
def test_indices(nx, ny, nz):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    w = workloads.make_tiny(nx, ny, nz)
    w["wells"] = w["wells"][:1] + w["wells"][1:] * (nx * ny > 1)
    m = r2p.Model(w)
    x = torch.as_tensor(workloads.random_state(w, np.random.default_rng(nx), p_spread=5.0), device="cuda")
    J = r2p.Jacobian(m)
    J.assemble(x, m.initial_state(), 2.0)
    P = r2p.Cpr().setup(J, r2p.cpr_opts(px=min(nx, 4), py=min(ny, 4)))
    L = P.amg_levels()[:3]
    f = L[0]
    # the 7-point pattern
    i = np.arange(m.n)
    deg = 1 + sum(((c > 0).astype(int) + (c < d - 1)) for c, d in
                  ((i % nx, nx), (i // nx % ny, ny), (i // (nx * ny), nz)))
    assert f["n"] == m.n and np.array_equal(np.diff(f["rp"]), deg) and f["rp"][0] == 0
    for f, c in zip(L, L[1:]):
        agg = f["agg"]
        assert np.array_equal(np.unique(agg), np.arange(c["n"]))
        rows = np.repeat(np.arange(f["n"]), np.diff(f["rp"]))
        pairs = np.unique(agg[rows].astype(np.int64) * c["n"] + agg[f["col"]])
        assert np.array_equal(pairs % c["n"], c["col"])
        assert np.array_equal(np.diff(c["rp"]), np.bincount(pairs // c["n"], minlength=c["n"]))
