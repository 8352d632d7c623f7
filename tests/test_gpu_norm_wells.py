"""The scaled norm over more rows than its workgroups take in one pass, and
the well rows' assembly over their numbers of perforations.

The norm is a maximum over rows of three roundings each: 4 eps from NumPy's.
A well's sums run over 1 to 130 perforations (a wavefront takes 64 at a time)
under every control; b and the Jacobian against the oracle at 1e-12 of their
largest element, the bound of the general assembly test.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    return torch, r2p


@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (255, 1, 1), (64, 64, 127), (101, 83, 63)])
def test_norm_is_the_largest_row(nx, ny, nz):
    torch, r2p = _gpu()
    w = workloads.make_tiny(nx, ny, nz)
    w["wells"] = w["wells"][:1] + w["wells"][1:] * (nx * ny > 1)
    m = r2p.Model(w)
    g, c, dt = w["grid"], w["const"], 2.5
    rng = np.random.default_rng(nx)
    pv = g["dx"] * g["dy"] * g["dz"] * w["phi"] / c["alpha_c"]
    b = rng.standard_normal(2 * (m.n + m.nw)) * 1e-3
    for row in {0, m.n - 1, m.n // 2, m.n}:               # the largest at either end, the middle, a well
        v = b.copy()
        v[2 * row] = -3e9
        t = np.array([abs(q["target"]) or 1.0 for q in w["wells"]])
        ref = max((np.abs(v[:2 * m.n].reshape(-1, 2)) * dt / pv[:, None]).max(),
                  (np.abs(v[2 * m.n::2]) / t).max())
        got = m.residual_norm(torch.as_tensor(v, device="cuda"), dt)
        out = torch.zeros(1, dtype=torch.float64, device="cuda")
        m.residual_norm_noalloc(torch.as_tensor(v, device="cuda"), dt, out)
        assert abs(got - ref) <= 4 * np.finfo(float).eps * ref
        assert float(out) == got
    for row in (0, 2 * m.n - 1, 2 * m.n):
        v = b.copy()
        v[row] = np.nan
        assert np.isnan(m.residual_norm(torch.as_tensor(v, device="cuda"), dt))


@pytest.mark.parametrize("control", [0, 1, 2, 3])
@pytest.mark.parametrize("nz", [1, 63, 64, 65, 130])
def test_well_rows(nz, control):
    torch, r2p = _gpu()
    import oracle
    oracle.build(force=False)
    w = workloads.make_tiny(3, 2, nz)
    w["wells"][1] = dict(w["wells"][1], ctrl=control)
    x = workloads.random_state(w, np.random.default_rng(nz))
    xo = workloads.random_state(w, np.random.default_rng(nz + 1))
    Jo, Fo = oracle.Model(w).jacobian(x, xo, 3.0)
    m = r2p.Model(w)
    J = r2p.Jacobian(m)
    b = J.assemble(torch.as_tensor(x, device="cuda"), torch.as_tensor(xo, device="cuda"), 3.0).cpu().numpy()
    assert np.abs(b + Fo).max() <= 1e-12 * np.abs(Fo).max()
    assert np.abs(b[2 * m.n:] + Fo[2 * m.n:]).max() <= 1e-12 * np.abs(Fo[2 * m.n:]).max()
    rp, col, val = J.export()
    assert np.array_equal(rp, Jo.rp) and np.array_equal(col, Jo.col)
    assert np.abs(val - Jo.val).max() <= 1e-12 * np.abs(Jo.val).max()
    lo = rp[m.n]
    assert np.abs(val[lo:] - Jo.val[lo:]).max() <= 1e-12 * np.abs(Jo.val[lo:]).max()
