"""A singular coarsest AMG matrix: an error, and the handle works afterwards.

A closed box of incompressible fluids in incompressible rock leaves the
pressure undetermined.  On a uniform chain the undecoupled pressure matrix is
t [1 -1; -1 2 -1; ..; -1 1], whose elimination has every multiplier exactly -1
and the last pivot exactly zero, where the blocked LU stops with the rows from
there on not chosen.  Overlap 0 cuts the chain for the RAS stage, so that its
subdomain matrices are regular.  The chains end in the first panel of 32
columns, at its edge, in the third one and in the last of 16 and 8 columns.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

ESINGULAR = -6


def _closed(nx):
    w = workloads.make_1d(nx)
    w["wells"] = []
    return w


def _state(m, nx):
    import torch
    x = m.initial_state()
    x[0::2] += torch.as_tensor(np.random.default_rng(nx).normal(0.0, 20.0, nx), device="cuda")
    x[1::2] = 0.5
    return x


def _opts(r2p, **kw):
    return r2p.cpr_opts(decouple=r2p.DEC_NONE, px=2, py=1, overlap=0, max_levels=1, **kw)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nx", [2, 4, 32, 33, 70, 1040, 2056])
def test_setup_reports_it_and_the_handle_recovers(nx, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    P = r2p.Cpr()
    m = r2p.Model(_closed(nx))
    x = _state(m, nx)
    J = r2p.Jacobian(m)
    J.assemble(x, x, 1.0)
    with pytest.raises(r2p.R2PError) as e:
        P.setup(J, _opts(r2p, precision=precision))
    assert e.value.code == ESINGULAR and "coarsest AMG matrix" in str(e.value)
    w2 = workloads.make_1d(nx)
    m2 = r2p.Model(w2)
    x2 = m2.initial_state()
    J2 = r2p.Jacobian(m2)
    b = J2.assemble(x2, x2, 1.0)
    P.setup(J2, r2p.cpr_opts(px=1, py=1, max_levels=1, precision=precision))
    _, info = r2p.solve(J2, P, b)
    assert info.status == 0


@pytest.mark.parametrize("nx", [2, 4])
def test_newton_step_ends_unconverged(nx):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    m = r2p.Model(_closed(nx))
    x = _state(m, nx)
    o = r2p.newton_opts()
    o.cpr = _opts(r2p)
    info = m.newton_step(x, 1.0, o)
    assert info.status == r2p.NOT_CONVERGED and info.setup_status == ESINGULAR
