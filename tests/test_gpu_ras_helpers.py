"""Prefetch helpers of the RAS sweep and the factorisation on wide levels.

Helper workgroups (subdomain counts that are multiples of 8) read ahead of a
sweep by the slice it is at, up to 128 slices of 32 rows (64 in the
factorisation).  A rough pressure field makes about one cell in seven a local
maximum, the first level and so the last of the backward sweep; a checkerboard
makes two levels of half the rows each, so that the factorisation's last one is
wide too.  A helper that was not told how far the sweep is inside such a level,
or that it is over, would wait for its spin bound.

Results: as in the layout test, against a level-by-level solve in NumPy.
Time: one wait that runs into the bound is 65,536 polls with sleeps of at least
512 cycles, 14 ms at 2.4 GHz; an application takes about 0.5 ms here and the
subdomains' part of a set-up some 3 ms, so both have to stay below 10 ms.
"""
import numpy as np
import pytest

import workloads
from test_gpu_ras_layout import test_factors_and_application as check_layout

pytestmark = pytest.mark.gpu

GRID = (160, 80, 32)
AHEAD = 32 * (128 + 8)       # rows


@pytest.mark.parametrize("precision", [0, 1])
def test_results_with_helpers(precision):
    check_layout(GRID + (4, 2, 1, 1, 50.0), precision)


def _state(w, kind):
    x = workloads.random_state(w, np.random.default_rng(1))
    if kind == "checkerboard":
        g = w["grid"]
        c = np.arange(g["n"])
        odd = (c % g["nx"] + c // g["nx"] % g["ny"] + c // (g["nx"] * g["ny"])) & 1
        x[0:2 * g["n"]:2] = w["const"]["p_ref"] + 50.0 * odd
    return x


@pytest.mark.parametrize("kind", ["random", "checkerboard"])
@pytest.mark.parametrize("precision", [0, 1])
def test_no_helper_waits_for_its_bound(kind, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    w = workloads.make_tiny(*GRID)
    m = r2p.Model(w)
    x = torch.as_tensor(_state(w, kind), device="cuda")
    J = r2p.Jacobian(m)
    J.assemble(x, m.initial_state(), 2.0)
    P = r2p.Cpr().setup(J, r2p.cpr_opts(px=4, py=2, precision=precision))
    width = np.bincount(P.ras_subdomain(0)["level"])
    assert width[0] > AHEAD
    if kind == "checkerboard":
        assert width[1] > AHEAD
    r = torch.randn(m.N, dtype=torch.float64, device="cuda")
    y = m.tensor()
    times = []
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        P.ras_apply(r, y)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    o = r2p.newton_opts(max_newton=1, cpr=P.opts, lin=r2p.solve_opts(maxit=1))
    setup = [m.newton_step(x.clone(), 2.0, o).ms_ras_setup for _ in range(3)]
    print(f"{kind} fp{64 >> precision}: application {min(times):.3f} ms, set-up {min(setup):.2f} ms")
    assert min(times) < 10.0 and min(setup) < 10.0


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("px,py", [(1, 1), (3, 1), (4, 3), (8, 8), (11, 8), (16, 8)])
def test_results_over_subdomain_counts(px, py, precision):
    """Helpers for counts that are no multiple of 8, two each, and none."""
    check_layout((64, 48, 30 if px * py < 16 else 6, px, py, 1, 1, 50.0), precision)


@pytest.mark.parametrize("precision", [0, 1])
def test_many_subdomains_are_not_held_up(precision):
    """128 subdomains have half the levels' work each of 64: on a smooth field
    one application takes no longer than with 64 (15% and 20 us for noise).
    One helper each, always late, once made it twice as long."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1701_06254_amd import r2p
    w = workloads.make_tiny(160, 80, 64)
    m = r2p.Model(w)
    x0 = m.initial_state()
    x = torch.as_tensor(workloads.developed_state(w, x0.cpu().numpy(), np.random.default_rng(0)),
                        device="cuda")
    r = torch.randn(m.N, dtype=torch.float64, device="cuda")
    y = m.tensor()
    best = {}
    for px, py in ((8, 8), (16, 8)):
        J = r2p.Jacobian(m)
        J.assemble(x, x0, 1.0)
        P = r2p.Cpr().setup(J, r2p.cpr_opts(px=px, py=py, precision=precision))
        times = []
        for _ in range(30):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            P.ras_apply(r, y)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        best[px * py] = min(times)
    print({k: f"{1e3 * v:.0f} us" for k, v in best.items()})
    assert best[128] <= 1.15 * best[64] + 0.02
