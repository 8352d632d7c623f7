"""Device memory that a preconditioner handle holds once it has solved.

The set-up of the factors needs one factor-sized array beside them (32 bytes
for each of a position's four main entries).  It shares the memory of the
Krylov basis, which is empty then, so the first solve adds at most the basis,
its preconditioned vectors and a few vectors, less that array.  Allocations are
rounded up, by 2 MiB at most each; about a dozen are made.
"""
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [8, 30])
@pytest.mark.parametrize("precision", [0, 1])
def test_first_solve_reuses_the_setup_array(restart, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    m = r2p.Model(workloads.make_tiny(100, 90, 60))
    x = m.initial_state()
    J = r2p.Jacobian(m)
    b = J.assemble(x, x, 1.0)
    y = m.tensor()
    P = r2p.Cpr().setup(J, r2p.cpr_opts(px=2, py=2, precision=precision))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    _, info = r2p.solve(J, P, b, r2p.solve_opts(restart=restart, maxit=2), y)
    torch.cuda.synchronize()
    added = before - torch.cuda.mem_get_info()[0]
    vectors = 2 * restart + 1 + 2
    shared = 32 * 4 * m.n
    assert added <= 8 * m.N * vectors - min(shared, 8 * m.N * (restart + 1)) + 12 * 2 ** 21
    # and it is what a second set-up and solve run on
    J.assemble(x, x, 1.0)
    P.setup(J, P.opts)
    r2p.solve(J, P, b, r2p.solve_opts(restart=restart, maxit=2), y)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= added + 2 ** 21
