"""What a program of this simulator does, as cases that can be timed and checked.

A case is one call (or the few calls that belong together) of the public
entry points in `paper_1701_06254_amd.r2p`, on a seeded synthetic reservoir
or network input:

  newton    one implicit time step: Newton's method with CPR-preconditioned
            solves (what a simulation run repeats);
  solve     one preconditioned Krylov solve of a Newton system whose
            preconditioner is set up;
  setup     assembly, CPR set-up and one application (what every Newton
            iteration does around its solve);
  cpr, ras, amg
            one application of the preconditioner, of its second stage (block
            ILU(0) in restricted additive Schwarz) or of one AMG cycle;
  assemble  residual, Jacobian and the scaled norm of the stopping test;
  spmv      one product with the Jacobian;
  forward   the warm-start network on a whole grid;
  train     loss and parameter gradient of the network on a batch of crops.

The reservoirs follow the repository's correlated-permeability workload:
ln k_h = 4.6 + G with a correlation length of about ten cells, k_z = 0.1 k_h,
porosity U(0.1, 0.3), vertical wells 40 columns apart (rate injectors and BHP
producers, checkerboard); the smallest is its 2,000-cell quarter five-spot.
The states have pressure mounds and sinks around the wells and water plumes
around the injectors, as some days into a run.
"""
import math

import numpy as np
import torch

from paper_1701_06254_amd import r2p

CONST = dict(beta_c=0.001127, alpha_c=5.614583, rho_o=46.244, rho_w=62.238, p_ref=4800.0,
             z_ref=8400.0, c_o=1e-5, c_w=1e-5, c_r=1e-5, mu_o=5.0, mu_w=1.0, grav=1.0)
DX, DY, DZ, TOP = 20.0, 20.0, 2.0, 8335.0
INJ, PROD, BHP, WRATE, LRATE = 0, 1, 0, 1, 3
SIGMA = 1.0      # standard deviation of ln k
RADIUS = 10.0    # mean radius of a water plume, cells
MOUND = 10.0     # psi above (below) hydrostatic at an injector (a producer)


def listed():
    return [
        # the smallest whole step: the 2,000-cell quarter five-spot at its
        # 10-day step, where launches and read-backs are the time
        dict(name="newton 20x20x5", op="newton", nx=20, ny=20, nz=5, spot=True, dt=10.0),
        # the benchmark model's step with the FP32 preconditioner
        dict(name="newton 200x200x50 fp32", op="newton", nx=200, ny=200, nz=50, dt=0.2, fp32=True),
        # one CPR-FGMRES(30) solve of a 2M-cell system, to the tolerance of
        # inexact Newton (the lower forcing bound, the paper's 1e-2)
        dict(name="solve 200x200x50", op="solve", nx=200, ny=200, nz=50, dt=0.1, rtol=0.01),
        # a model of some ten thousand cells with odd extents, Algorithm 2 and
        # overlap 2 (the paper's own variants)
        dict(name="solve 61x47x13 fpf", op="solve", nx=61, ny=47, nz=13, dt=0.2, form=1, overlap=2),
        # what a Newton iteration at 2M cells does beside its solve
        dict(name="setup 200x200x50", op="setup", nx=200, ny=200, nz=50, dt=1.6),
        # the second stage alone with the benchmark's 16 subdomains
        dict(name="ras 200x200x50", op="ras", nx=200, ny=200, nz=50, dt=1.6),
        # the preconditioner in the large model's form (one subdomain per CU,
        # one K-cycle on two levels) at 8.2M cells, the largest case
        dict(name="cpr 320x320x80 16x16", op="cpr", nx=320, ny=320, nz=80, dt=0.4, px=16, py=16,
             kcycle=2, cycles=1),
        # one AMG cycle of a mid-size model with odd extents
        dict(name="amg 83x101x29", op="amg", nx=83, ny=101, nz=29, dt=0.8),
        # the Newton loop's assembly and stopping test at 2M cells
        dict(name="assemble 200x200x50", op="assemble", nx=200, ny=200, nz=50, dt=0.8),
        # one product with the Jacobian, odd extents
        dict(name="spmv 173x181x37", op="spmv", nx=173, ny=181, nz=37, dt=0.8),
        # the warm start's inference on the benchmark grid
        dict(name="forward 1x50x200x200", op="forward", nb=1, nz=50, ny=200, nx=200),
        # one training step's gradient: four 48x48-column crops of 50 layers,
        # the batch of the training loop
        dict(name="train 4x50x48x48", op="train", nb=4, nz=50, ny=48, nx=48),
    ]


# The most cells (voxels) of a drawn case, by operation: each stays below the
# largest listed case of its kind.
MOST = dict(newton=300_000, solve=1_500_000, setup=1_900_000, ras=1_900_000, cpr=4_000_000,
            amg=4_000_000, assemble=4_000_000, spmv=4_000_000, forward=1_900_000, train=440_000)


def draw(rng):
    op = rng.choice(sorted(MOST))
    if op in ("forward", "train"):
        n = math.exp(rng.uniform(math.log(4_000), math.log(MOST[op])))
        nb = rng.choice([1, 1, 2, 4]) if op == "train" else 1
        nz = rng.randint(4, 50)
        side = max(8.0, math.sqrt(n / nb / nz))
        r = rng.uniform(0.7, 1.4)
        return dict(op=op, nb=nb, nz=nz, ny=max(4, int(side * r)), nx=max(4, int(side / r)))
    n = math.exp(rng.uniform(math.log(2_000), math.log(MOST[op])))
    nz = rng.randint(3, 12) if n < 40_000 else rng.randint(10, 60)
    side = max(16.0, math.sqrt(n / nz))
    r = rng.uniform(0.7, 1.4)
    most = 0.1 if op == "solve" else 0.4
    c = dict(op=op, nx=max(16, int(side * r)), ny=max(16, int(side / r)), nz=nz,
             dt=round(math.exp(rng.uniform(math.log(0.03), math.log(most))), 3))
    if op in ("assemble", "spmv"):
        return c
    # options in earnest use: Algorithm 2, overlap, tile counts, the V-cycle
    # and the cycle counts, the FP32 preconditioner inside Newton's method
    if rng.random() < 0.25:
        c["form"] = 1
    if rng.random() < 0.2:
        c["overlap"] = 2
    t = rng.choice([4, 4, 4, 2, 8])
    if t != 4 and min(c["nx"], c["ny"]) >= 4 * t and (t > 2 or n < 200_000):
        c["px"] = c["py"] = t
    if rng.random() < 0.25:
        c["kcycle"] = rng.choice([0, 2])
    if rng.random() < 0.25:
        c["cycles"] = rng.choice([1, 3])
    if op == "newton" and rng.random() < 0.5:
        c["fp32"] = True
    if op == "solve":
        if n > 20_000:
            c["rtol"] = rng.choice([0.1, 0.01, 0.01])
        if rng.random() < 0.25:
            c["restart"] = rng.choice([20, 40])
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _field(shape, g, corr=10):
    """A standardised correlated field on (nz, ny, nx): coarse Gaussian noise
    interpolated to the grid."""
    coarse = [max(2, -(-s // corr) + 1) for s in shape]
    z = torch.randn([1, 1] + coarse, generator=g, device="cuda", dtype=torch.float64)
    f = torch.nn.functional.interpolate(z, size=shape, mode="trilinear", align_corners=True)[0, 0]
    return ((f - f.mean()) / f.std()).contiguous()


def _lattice(c):
    """(i, j, kind, control, target) of every well."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    if c.get("spot"):
        return [(0, 0, INJ, WRATE, 200.0), (nx - 1, ny - 1, PROD, LRATE, 200.0)]
    a, b = max(2, round(nx / 40)), max(1, round(ny / 40))
    out = []
    for p in range(a):
        for q in range(b):
            i, j = int((p + 0.5) * nx / a), int((q + 0.5) * ny / b)
            out.append((i, j, INJ, WRATE, 80.0 * nz) if (p + q) % 2 == 0
                       else (i, j, PROD, BHP, 4000.0))
    return out


def _reservoir(c, seed):
    """Rock fields (device, natural order), the wells, and the state at the
    start of a step."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    n = nx * ny * nz
    g = _gen(seed)
    if c.get("spot"):
        kh = torch.exp(4.6 + torch.randn(n, generator=g, device="cuda", dtype=torch.float64))
        kz = kh.clone()
        phi = 0.15 + 0.1 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    else:
        kh = torch.exp(4.6 + SIGMA * _field((nz, ny, nx), g)).reshape(-1)
        kz = 0.1 * kh
        phi = 0.1 + 0.2 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    wells = _lattice(c)
    nw = len(wells)
    x = torch.zeros(2 * (n + nw), dtype=torch.float64, device="cuda")
    depth = TOP + DZ * torch.arange(nz, device="cuda", dtype=torch.float64)
    p = (CONST["p_ref"] + CONST["rho_o"] / 144.0 * (depth - CONST["z_ref"]))[:, None, None]
    p = p.expand(nz, ny, nx).clone()
    s = torch.zeros_like(p)
    if not c.get("spot"):
        ii = torch.arange(nx, device="cuda", dtype=torch.float64)
        jj = torch.arange(ny, device="cuda", dtype=torch.float64)
        for i, j, kind, _, _ in wells:
            r = torch.hypot(ii[None, :] - i, jj[:, None] - j)
            p += (MOUND if kind == INJ else -MOUND) * torch.exp(-r / 15.0)[None]
            if kind == INJ:
                ph = 6.28 * torch.rand(1, generator=g, device="cuda", dtype=torch.float64)
                R = RADIUS * (1.0 + 0.4 * torch.sin(ph + 6.28 * (depth - TOP) / (DZ * nz)))
                s = torch.maximum(s, 0.8 * (1.0 - r[None] / R[:, None, None]).clamp(0.0, 1.0))
    x[0:2 * n:2] = p.reshape(-1)
    x[1:2 * n:2] = s.reshape(-1)
    for k, (i, j, kind, ctrl, target) in enumerate(wells):
        top = p[0, j, i]
        x[2 * (n + k)] = target if ctrl == BHP else top + (100.0 if kind == INJ else -100.0)
    return dict(kx=kh, ky=kh, kz=kz, phi=phi, wells=wells, n=n, x=x, g=g)


def _model(c, res):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    kh, kz, phi = (res[k].cpu().numpy() for k in ("kx", "kz", "phi"))
    wells = [dict(cells=np.array([i + nx * (j + ny * k) for k in range(nz)], dtype=np.int32),
                  kind=kind, ctrl=ctrl, target=target, rw=0.25, skin=0.0)
             for i, j, kind, ctrl, target in res["wells"]]
    return r2p.Model(dict(grid=dict(nx=nx, ny=ny, nz=nz, n=res["n"], dx=DX, dy=DY, dz=DZ, top=TOP),
                          kx=kh, ky=kh, kz=kz, phi=phi, wells=wells, const=CONST))


def _iterate(c, res):
    """A Newton iterate inside a step from the state: the pressure moved by a
    smooth field of a few psi, the saturation inside the plumes by a few
    percent."""
    n, x, g = res["n"], res["x"].clone(), res["g"]
    shape = (c["nz"], c["ny"], c["nx"])
    x[0:2 * n:2] += 2.0 * _field(shape, g).reshape(-1)
    s = x[1:2 * n:2]
    ds = 0.02 * _field(shape, g).reshape(-1)
    x[1:2 * n:2] = torch.where(s > 0.0, (s + ds).clamp(0.0, 1.0), s)
    return x


def _vector(size, res):
    return torch.randn(size, generator=res["g"], device="cuda", dtype=torch.float64)


def _cpr_opts(c):
    return r2p.cpr_opts(form=c.get("form", 0), px=c.get("px", 4), py=c.get("py", 4),
                        overlap=c.get("overlap", 1), precision=r2p.FP32 if c.get("fp32") else r2p.FP64,
                        kcycle=c.get("kcycle", 1), amg_cycles=c.get("cycles", 2))


BLOCKS, CH, NIN, NOUT = 4, 32, 6, 2


def _network(c, seed):
    """Parameters (the library's compact order), features and targets."""
    g = _gen(seed)
    V = c["nb"] * c["nz"] * c["ny"] * c["nx"]
    dims = [(NIN, CH)] + [(CH, CH)] * (2 * BLOCKS) + [(CH, NOUT)]
    theta = []
    for l, (cin, cout) in enumerate(dims):
        std = math.sqrt(2.0 / (27 * cin)) * (0.5 if l and l % 2 == 0 else 1.0)
        theta.append(std * torch.randn(27 * cout * cin, generator=g, device="cuda"))
        theta.append(0.05 * torch.randn(cout, generator=g, device="cuda"))
    feat = torch.zeros(V, CH, device="cuda", dtype=torch.bfloat16)
    feat[:, :NIN] = torch.randn(V, NIN, generator=g, device="cuda").to(torch.bfloat16)
    tgt = torch.randn(V, NOUT, generator=g, device="cuda")
    return torch.cat(theta), feat, tgt


def prepare(case, seed):
    op = case["op"]
    if op in ("forward", "train"):
        theta, feat, tgt = _network(case, seed)
        net = r2p.Cnn(blocks=BLOCKS)
        net.set_params(theta.cpu().numpy())
        V = feat.shape[0]
        return dict(op=op, net=net, feat=feat.view(torch.int16), tgt=tgt.reshape(-1),
                    shape=(case["nb"], case["nz"], case["ny"], case["nx"]),
                    out=torch.empty(2 * V, dtype=torch.float32, device="cuda"))
    res = _reservoir(case, seed)
    m = _model(case, res)
    st = dict(op=op, model=m, x=res["x"], dt=case["dt"])
    if op == "newton":
        st["opts"] = r2p.newton_opts(cpr=_cpr_opts(case))
        return st
    st["xk"] = _iterate(case, res)
    st["J"] = J = r2p.Jacobian(m)
    st["b"] = b = m.tensor()
    st["y"] = m.tensor()
    if op == "assemble":
        return st
    if op == "spmv":
        st["v"] = _vector(m.N, res)
        J.assemble(st["xk"], st["x"], st["dt"], b)
        return st
    st["P"] = P = r2p.Cpr()
    st["copts"] = _cpr_opts(case)
    if op == "setup":
        return st
    J.assemble(st["xk"], st["x"], st["dt"], b)
    P.setup(J, st["copts"])
    if op == "solve":
        st["sopts"] = r2p.solve_opts(restart=case.get("restart", 30), rtol=case.get("rtol", 1e-8))
    else:
        st["v"] = _vector(m.n if op == "amg" else m.N, res)
        if op == "amg":
            st["y"] = m.tensor(m.n)
    return st


def run(state):
    op = state["op"]
    if op == "newton":
        x = state["x"].clone()
        info = state["model"].newton_step(x, state["dt"], state["opts"])
        return dict(x=x, status=int(info.status))
    if op == "solve":
        y, info = r2p.solve(state["J"], state["P"], state["b"], state["sopts"], state["y"])
        return dict(y=y, status=int(info.status))
    if op == "setup":
        J, P = state["J"], state["P"]
        J.assemble(state["xk"], state["x"], state["dt"], state["b"])
        P.setup(J, state["copts"])
        return dict(z=P.apply(state["b"], state["y"]))
    if op == "cpr":
        return dict(z=state["P"].apply(state["v"], state["y"]))
    if op == "ras":
        return dict(z=state["P"].ras_apply(state["v"], state["y"]))
    if op == "amg":
        return dict(z=state["P"].amg_vcycle(state["v"], state["y"]))
    if op == "assemble":
        b = state["J"].assemble(state["xk"], state["x"], state["dt"], state["b"])
        return dict(b=b, norm=state["model"].residual_norm(b, state["dt"]))
    if op == "spmv":
        return dict(y=state["J"].spmv(state["v"], state["y"]))
    if op == "forward":
        return dict(out=state["net"].forward(state["feat"], state["shape"], state["out"]))
    loss = state["net"].backward(state["feat"], state["tgt"], state["shape"])
    return dict(loss=loss, grads=state["net"].get_grads())


# -------------------------------------------------------------------- work
def work(case):
    """Each input read once and each output written once.  Per cell: the
    Jacobian's seven 2x2 blocks 224 bytes, a state or residual pair 16; the
    factors of the second stage hold the same blocks with overlap."""
    op = case["op"]
    n = case["nx"] * case["ny"] * case["nz"]
    if op in ("forward", "train"):
        V = n * case["nb"]
        flops = 2 * 27 * (NIN * CH + 2 * BLOCKS * CH * CH + CH * NOUT) * V
        # every layer's activations written and read once in bfloat16
        act = 2 * CH * V * (2 * BLOCKS + 2)
        return dict(bytes=(2 if op == "forward" else 4) * act + 8 * V,
                    flops=flops * (1 if op == "forward" else 3))
    flops = dict(spmv=56, assemble=900, amg=120, ras=110, cpr=350, setup=1500, solve=400,
                 newton=2400)[op] * n
    fields = 32 * n                                    # tx, ty, tz, porosity
    by = dict(spmv=224 + 32, assemble=224 + 48, amg=56 + 16, ras=224 + 32, cpr=224 + 56 + 32,
              setup=224 + 224 + 80, solve=224 + 224 + 32, newton=32 + 224)[op] * n
    return dict(bytes=by + (fields if op in ("assemble", "setup", "newton") else 0), flops=flops)


# ------------------------------------------------- the same in plain torch
def _residual(c, res, dt):
    """F(x) of the discrete two-phase system for a step from res['x'], in
    plain torch: accumulation, upwinded two-point fluxes with gravity,
    Peaceman wells."""
    nx, ny, nz, n, wells = c["nx"], c["ny"], c["nz"], res["n"], res["wells"]
    C = CONST
    shape = (nz, ny, nx)
    kx, ky, kz, phi = (res[k].reshape(shape) for k in ("kx", "ky", "kz", "phi"))

    def harmonic(k, axis, d, area):
        a, b = k.narrow(axis, 0, k.shape[axis] - 1), k.narrow(axis, 1, k.shape[axis] - 1)
        return area / (d / (2.0 * a) + d / (2.0 * b))

    faces = [(0, harmonic(kz, 0, DZ, DX * DY), DZ), (1, harmonic(ky, 1, DY, DX * DZ), 0.0),
             (2, harmonic(kx, 2, DX, DY * DZ), 0.0)]
    coef = DX * DY * DZ / (C["alpha_c"] * dt)
    phases = [(C["rho_o"], C["c_o"], C["mu_o"], lambda s: (1.0 - s) ** 2),
              (C["rho_w"], C["c_w"], C["mu_w"], lambda s: s ** 2)]
    kzw = torch.arange(nz, device=kx.device)
    depth = TOP + DZ * kzw.to(torch.float64)

    def split(x):
        return x[0:2 * n:2].reshape(shape), x[1:2 * n:2].reshape(shape)

    def mass(p, s):
        por = phi * (1.0 + C["c_r"] * (p - C["p_ref"]))
        return [por * (1.0 + cc * (p - C["p_ref"])) * (1.0 - s if a == 0 else s)
                for a, (_, cc, _, _) in enumerate(phases)]

    old = mass(*split(res["x"]))

    def F(x):
        p, s = split(x)
        out, well_rows = [], []
        perf = []
        for k, (i, j, kind, ctrl, target) in enumerate(wells):
            ro = 0.28 * math.sqrt(DX * DX + DY * DY) / 2.0
            WI = 2.0 * math.pi * C["beta_c"] * kx[:, j, i] * DZ / math.log(ro / 0.25)
            pc, sc, pb = p[:, j, i], s[:, j, i], x[2 * (n + k)]
            lam = [kr(sc) * (1.0 + cc * (pc - C["p_ref"])) / mu for _, cc, mu, kr in phases]
            dp = [pb - pc - rho * (1.0 + cc * (pc - C["p_ref"])) / 144.0 * (depth[0] - depth)
                  for rho, cc, _, _ in phases]
            if kind == INJ:
                q = [torch.zeros_like(pc), WI * (lam[0] + lam[1]) * dp[1]]
            else:
                q = [WI * lam[0] * dp[0], WI * lam[1] * dp[1]]
            perf.append((i, j, q))
            sign = 1.0 if kind == INJ else -1.0
            if ctrl == BHP:
                well_rows.append(pb - target)
            elif ctrl == WRATE:
                well_rows.append(q[1].sum() - sign * target)
            else:
                well_rows.append((q[0] + q[1]).sum() - sign * target)
            well_rows.append(x[2 * (n + k) + 1])
        for a, (rho, cc, mu, kr) in enumerate(phases):
            b = 1.0 + cc * (p - C["p_ref"])
            gam = C["grav"] * rho * b / 144.0
            lam = kr(s) * b / mu
            f = coef * (mass(p, s)[a] - old[a])
            for axis, tg, dz in faces:
                m = p.shape[axis] - 1
                if m < 1:
                    continue
                lo = lambda t: t.narrow(axis, 0, m)  # noqa: E731
                hi = lambda t: t.narrow(axis, 1, m)  # noqa: E731
                dphi = (hi(p) - lo(p)) - 0.5 * (lo(gam) + hi(gam)) * dz
                flux = C["beta_c"] * tg * torch.where(dphi >= 0.0, hi(lam), lo(lam)) * dphi
                pad = [0, 0] * 3
                pad[2 * (2 - axis) + 1] = 1
                into_lo = torch.nn.functional.pad(flux, pad)
                pad = [0, 0] * 3
                pad[2 * (2 - axis)] = 1
                f = f - into_lo + torch.nn.functional.pad(flux, pad)
            src = torch.zeros(nz, ny * nx, dtype=torch.float64, device=kx.device)
            if perf:
                cols = torch.tensor([j * nx + i for i, j, _ in perf], device=kx.device)
                src = src.index_add(1, cols, torch.stack([q[a] for _, _, q in perf], 1))
            out.append((f - src.reshape(shape)).reshape(-1))
        cells = torch.stack(out, 1).reshape(-1)
        return torch.cat([cells, torch.stack(well_rows)]) if well_rows else cells

    return F


def _dense(F, x):
    """dF/dx as a dense matrix, its columns by forward mode."""
    cols = torch.func.vmap(lambda v: torch.func.jvp(F, (x,), (v,))[1], chunk_size=512)
    return cols(torch.eye(x.numel(), dtype=x.dtype, device=x.device)).t().contiguous()


def _scaled_norm(c, res, f, dt):
    n = res["n"]
    pv = DX * DY * DZ * res["phi"] / CONST["alpha_c"]
    v = (f[:2 * n].reshape(n, 2).abs() * dt / pv[:, None]).max()
    for k, w in enumerate(res["wells"]):
        v = torch.maximum(v, f[2 * (n + k)].abs() / abs(w[4]))
    return float(v)


def _conv(x, w, b):
    """3x3x3 convolution with zero padding in 64 bits: x [nb,nz,ny,nx,cin],
    w [27,cout,cin]."""
    nb, nz, ny, nx, cin = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    out = b.expand(nb * nz * ny * nx, w.shape[1])
    for t in range(27):
        dz, dy, dx = t // 9, t // 3 % 3, t % 3
        a = xp[:, dz:dz + nz, dy:dy + ny, dx:dx + nx].reshape(-1, cin)
        out = out + a @ w[t].t().contiguous()
    return out.reshape(nb, nz, ny, nx, -1)


def _net64(case, theta, feat):
    dims = [(NIN, CH)] + [(CH, CH)] * (2 * BLOCKS) + [(CH, NOUT)]
    at, lay = 0, []
    for cin, cout in dims:
        w = theta[at:at + 27 * cout * cin].reshape(27, cout, cin)
        at += 27 * cout * cin
        lay.append((w, theta[at:at + cout]))
        at += cout
    h = feat[:, :NIN].double().reshape(case["nb"], case["nz"], case["ny"], case["nx"], NIN)
    h = torch.relu(_conv(h, *lay[0]))
    for k in range(BLOCKS):
        h = h + _conv(torch.relu(_conv(h, *lay[1 + 2 * k])), *lay[2 + 2 * k])
    return _conv(h, *lay[-1]).reshape(-1)


def exact(case, seed):
    op = case["op"]
    if op in ("forward", "train"):
        theta, feat, tgt = _network(case, seed)
        theta = theta.double()
        if op == "forward":
            with torch.no_grad():
                return dict(out=_net64(case, theta, feat))
        theta.requires_grad_(True)
        out = _net64(case, theta, feat)
        loss = ((out - tgt.reshape(-1).double()) ** 2).mean()
        return dict(loss=float(loss.detach()), grads=torch.autograd.grad(loss, theta)[0])
    if op in ("cpr", "ras", "amg", "setup"):
        return None      # a preconditioner's value is fixed by its own algorithm
    res = _reservoir(case, seed)
    F, dt = _residual(case, res, case["dt"]), case["dt"]
    if op == "newton":
        if 2 * res["n"] > 4000:
            return None  # a dense solve per iteration
        x = res["x"].clone()
        N2 = 2 * res["n"]
        sat = torch.arange(x.numel(), device=x.device)
        sat = (sat % 2 == 1) & (sat < N2)
        for _ in range(60):
            f = F(x)
            if _scaled_norm(case, res, f, dt) <= 1e-12:
                break
            y = torch.linalg.solve(_dense(F, x), -f)
            y = torch.where(sat, y.clamp(-0.2, 0.2), y)
            x = x + y
            x = torch.where(sat, x.clamp(0.0, 1.0), x)
        return dict(x=x, status=None)
    xk = _iterate(case, res)
    if op == "assemble":
        f = F(xk)
        return dict(b=-f, norm=_scaled_norm(case, res, f, dt))
    if op == "spmv":
        v = _vector(2 * (res["n"] + len(res["wells"])), res)
        return dict(y=torch.func.jvp(F, (xk,), (v,))[1])
    if res["n"] > 6000:
        return None      # a dense solve
    return dict(y=torch.linalg.solve(_dense(F, xk), -F(xk)), status=None)
