"""Performance cases of the Richards solver's public entry points.

Each case is one call (or one short run) that a program using the library
makes, on synthetic heterogeneous soils: lognormal K_s on a box, the Haverkamp
laws, a wet top face over dry soil.  Sizes span what the recipes, the serving
stream and the benchmark use: 16^3 to 256^3 cells, odd boxes and thin slabs,
FP64 and mixed precision, the three interface means.

Kinds
  residual  theta(p) and Phi(p) of a state (a user's own time loop or check)
  rebuild   J, M and the preconditioner at a new state, each applied once
  vcycle    one preconditioner application
  gmres     one Newton correction solved to eta
  step      one backward-Euler step of a resident simulation
  simulate  a whole short simulation: create, set-up, steps, result
  serve     a burst of requests through the ensemble server
"""
import math
from types import SimpleNamespace

import torch

import paper_2112_05051_amd as rich

KS0, P_INIT, P_TOP = 0.00944, -61.5, -20.7  # cm/s, cm, cm
LAWS = dict(alpha=1.611e6, beta=3.96, theta_s=0.287, theta_r=0.075, A=1.175e6, gamma=4.74)
MEANS = {"arith": 0, "upstream": 1, "harmonic": 2}


def _case(kind, nx, ny, nz, **kw):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, mean="arith", mixed=True, sigma=2.0, ell=8.0, dt=10.0, thin=False,
             levels=10, msbset=10, steps=1, requests=0, active=0)
    c.update(kw)
    return c


def listed():
    cases = [
        # a check of one small state, as the unit of a parameter study makes it: latency
        _case("residual", 16, 16, 16, name="residual_16", mean="harmonic", mixed=False, sigma=0.0, dt=1.0),
        # the residual of the benchmark's grid (one per line-search trial)
        _case("residual", 256, 256, 256, name="residual_256", mean="upstream", sigma=2.5, ell=16.0),
        # a new Jacobian on the benchmark's grid, every tenth Newton iteration or (msbset = 1) each one
        _case("rebuild", 256, 256, 256, name="rebuild_256_mixed", mean="upstream", sigma=2.5, ell=16.0),
        # the preconditioner alone: the benchmark's grid in single precision, an odd box in double
        _case("vcycle", 256, 256, 256, name="vcycle_256_mixed", mean="upstream", sigma=2.5, ell=16.0),
        _case("vcycle", 101, 67, 45, name="vcycle_101x67x45_fp64", mixed=False),
        # one linear solve of the FP64 recipe
        _case("gmres", 128, 128, 128, name="gmres_128_fp64", mixed=False),
        # the smallest recipe's time step: homogeneous, harmonic, two levels, FP64
        _case("step", 16, 16, 16, name="step_16_fp64", mean="harmonic", mixed=False, sigma=0.0, dt=1.0, levels=2),
        # an ensemble member's time step, the middle size of the serving stream
        _case("step", 64, 64, 64, name="step_64_mixed", mean="upstream", sigma=1.5, ell=4.0),
        # the paper's infiltration test on a quarter of its columns: thin grid, Dirichlet patch, GMRES(10)
        _case("step", 199, 199, 38, name="step_thin_199x199x38_mixed", mean="upstream", sigma=0.0, dt=2.0 / 9.0,
              thin=True),
        # the benchmark's time step with a fresh Jacobian every Newton iteration
        _case("step", 256, 256, 256, name="step_256_mixed_fresh_j", mean="upstream", sigma=2.5, ell=16.0, msbset=1),
        # a whole small simulation from nothing: allocation, AMG set-up, three steps
        _case("simulate", 48, 48, 48, name="simulate_48_mixed", sigma=1.5, ell=3.0, steps=3),
        # a burst of mixed-size requests on a resident server
        _case("serve", 32, 32, 32, name="serve_8_requests", sigma=1.5, ell=2.0, steps=2, requests=8, active=4),
    ]
    return cases


def _box(rng, lo, hi):
    """An odd box of about exp(U[log lo, log hi]) cells, aspect ratios 1/2..2."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    a, b = 2.0 ** rng.uniform(-1, 1), 2.0 ** rng.uniform(-1, 1)
    e = (n / (a * b)) ** (1.0 / 3.0)
    return tuple(max(4, int(round(v))) for v in (e * a, e * b, e))


def draw(rng):
    kind = rng.choice(["residual", "rebuild", "vcycle", "gmres", "step", "step", "simulate", "serve"])
    lo, hi = {"residual": (16 ** 3, 256 ** 3), "rebuild": (16 ** 3, 224 ** 3), "vcycle": (20 ** 3, 256 ** 3),
              "gmres": (16 ** 3, 128 ** 3), "step": (16 ** 3, 144 ** 3), "simulate": (16 ** 3, 56 ** 3),
              "serve": (14 ** 3, 36 ** 3)}[kind]
    nx, ny, nz = _box(rng, lo, hi)
    if kind in ("residual", "rebuild", "vcycle") and rng.random() < 0.2:  # the thin grids of the infiltration test
        return _case(kind, rng.randint(50, 398), rng.randint(50, 398), rng.randint(8, 38), thin=True, sigma=0.0,
                     dt=2.0 / 9.0, mean="upstream", mixed=rng.random() < 0.5)
    # the iteration's result in single precision carries its rounding: solves are compared in FP64
    mixed = kind != "gmres" and rng.random() < 0.6
    kw = dict(mean=rng.choice(["arith", "upstream"]), mixed=mixed, sigma=round(rng.uniform(1.0, 2.0), 2),
              ell=round(max(1.0, min(nx, ny, nz) * rng.uniform(0.04, 0.08)), 2))
    if kind == "step":
        kw["msbset"] = rng.choice([1, 10, 10])
    if kind == "simulate":
        kw["steps"] = rng.randint(1, 3)
    if kind == "serve":
        kw.update(steps=rng.randint(1, 2), requests=rng.randint(3, 8), active=rng.randint(2, 6))
    return _case(kind, nx, ny, nz, **kw)


# ------------------------------------------------------------------ inputs
def _problem(c, nx, ny, nz):
    if c["thin"]:
        h, top, wet = (64.0 / (nx + 1), 64.0 / (ny + 1), 1.0 / (nz + 1)), P_INIT, 5
        types = (1,) * 6
    else:
        h, top, wet = tuple(64.0 / (n + 1) for n in (nx, ny, nz)), P_TOP, -1
        types = (0, 0, 0, 0, 0, 1)
    return SimpleNamespace(nx=nx, ny=ny, nz=nz, hx=h[0], hy=h[1], hz=h[2], mean=MEANS[c["mean"]], dt=c["dt"],
                           bc_type=types, bc_value=(P_INIT if c["thin"] else 0.0,) * 5 + (top,), patch_face=wet,
                           patch_lo=(16.0, 16.0), patch_hi=(48.0, 48.0), patch_value=0.0, mean_vertical=-1, **LAWS)


def _options(c):
    """The recipes' solver controls."""
    thin = c["thin"]
    return SimpleNamespace(fnormtol=1e-8, scsteptol=2.220446049250313e-16 ** (2.0 / 3.0), max_newton=200, msbset=c["msbset"],
                           ls_alpha=1e-4, mxnewtstep=0.0, gmres_restart=10 if thin else 30,
                           eta=1e-7 if thin else 1e-6, gmres_maxit=200, amg_max_levels=c["levels"],
                           amg_coarse_size=512, amg_sweeps=3, coarse_dense_max=4096, coarse_l1_sweeps=4, amg_refresh=1,
                           precision=rich.PREC_MIXED if c["mixed"] else rich.PREC_FP64, gmres_reorth=0.01, aux_dflux=0,
                           amg_smoothed=0, tile_kz=0, smoother=0, amg_aggregation=0, amg_theta=0.0, amg_block=4096,
                           gmres_block=5 if thin else 10, gmres_shift=0.65, gmres_shift_span=0.55)


def _ks(c, nx, ny, nz, gen):
    """K_s0 exp(sigma Z), Z a smoothed normal field of unit variance (periodic), correlation ell/ell/(ell/4) cells."""
    n = nx * ny * nz
    if c["sigma"] == 0.0:
        # one soil, its conductivity uncertain
        return torch.full((n,), KS0, dtype=torch.float64, device="cuda") * math.exp(
            0.2 * float(torch.randn((), generator=gen, device="cuda", dtype=torch.float64)))
    z = torch.randn((nz, ny, nx), generator=gen, device="cuda", dtype=torch.float64)
    f = torch.fft.rfftn(z)
    for axis, (m, e) in enumerate(((nz, max(1.0, c["ell"] / 4)), (ny, c["ell"]), (nx, c["ell"]))):
        w = torch.fft.rfftfreq(m, device="cuda", dtype=torch.float64) if axis == 2 else torch.fft.fftfreq(
            m, device="cuda", dtype=torch.float64)
        f = f * torch.exp(-0.5 * (math.pi * e * w) ** 2).reshape([-1 if a == axis else 1 for a in range(3)])
    z = torch.fft.irfftn(f, s=(nz, ny, nx)).reshape(-1)
    z = (z - z.mean()) / z.std()
    return KS0 * torch.exp(c["sigma"] * z)


def _front(P, gen):
    """An infiltration front: wet above a rough depth, dry below, some cells saturated."""
    k = torch.arange(P.nz, device="cuda", dtype=torch.float64).reshape(-1, 1, 1) / P.nz
    depth = 0.7 + 0.1 * torch.randn((1, P.ny, P.nx), generator=gen, device="cuda", dtype=torch.float64)
    p = P_INIT + (P_TOP - P_INIT) * torch.sigmoid(20.0 * (k - depth))
    p = p + 0.5 * torch.randn((P.nz, P.ny, P.nx), generator=gen, device="cuda", dtype=torch.float64)
    if P.patch_face >= 0:
        p = torch.where((k > 0.9) & (depth > 0.8), torch.full_like(p, 0.5), p)
    return p.reshape(-1).contiguous()


def _inputs(c, seed):
    """(problem, options, K_s, state, a second random vector) of a single-simulation case."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    P = _problem(c, c["nx"], c["ny"], c["nz"])
    ks = _ks(c, P.nx, P.ny, P.nz, gen)
    p = _front(P, gen)
    x = torch.randn(p.shape, generator=gen, device="cuda", dtype=torch.float64)
    return P, _options(c), ks, p, x


def _requests(c, seed):
    """The server's requests: host arrays, sizes around the case's box, two means, all steps from the dry state."""
    reqs = []
    for r in range(c["requests"]):
        gen = torch.Generator(device="cuda").manual_seed(int(seed) * 64 + r)
        f = (0.75, 1.0, 1.25)[r % 3]
        nx, ny, nz = (max(4, int(round(v * f))) for v in (c["nx"], c["ny"], c["nz"]))
        d = dict(c, mean=("arith", "upstream")[r % 2])
        P = _problem(d, nx, ny, nz)
        ks = _ks(c, nx, ny, nz, gen).cpu().numpy()
        reqs.append((P, _options(d), ks, torch.full((nx * ny * nz,), P_INIT, dtype=torch.float64).numpy()))
    return reqs


def prepare(case, seed):
    c = case
    if c["kind"] == "serve":
        return SimpleNamespace(c=c, reqs=_requests(c, seed), server=rich.Server(64 << 30, c["active"]))
    P, O, ks, p, x = _inputs(c, seed)
    st = SimpleNamespace(c=c, P=P, O=O, ks=ks, p=p, x=x, solver=None)
    if c["kind"] == "simulate":
        st.p = torch.full_like(p, P_INIT)
        return st
    if c["kind"] == "residual":
        st.x = p + 0.5 * x  # a trial state near the previous level
    st.solver = rich.Solver(P, O, ks)
    if c["kind"] == "step":
        # a resident simulation after its first step (the AMG hierarchy is built there)
        st.solver.set_state(torch.full_like(p, P_INIT))
        st.solver.step(1)
        st.p = st.solver.get_state()
    elif c["kind"] in ("rebuild", "vcycle"):
        # the hierarchy's aggregates come from the dry state, as in a simulation; its values from the front
        st.solver.assemble(torch.full_like(p, P_INIT))
        st.solver.assemble(p)
    elif c["kind"] == "gmres":
        # the first Newton correction from the dry state: right-hand side -Phi(p0)
        st.p = torch.full_like(p, P_INIT)
        st.solver.assemble(st.p)
        st.x = -st.solver.residual(st.p, st.solver.theta(st.p)) * (1.0 + 0.1 * x)
    return st


def run(state):
    c = state.c
    kind = c["kind"]
    if kind == "serve":
        ids = [state.server.submit(P, O, ks, p0, c["steps"]) for P, O, ks, p0 in state.reqs]
        state.server.run_until_idle()
        return [state.server.poll(i)["p"] for i in ids]
    if kind == "simulate":
        s = rich.Solver(state.P, state.O, state.ks)
        s.set_state(state.p)
        s.step(c["steps"])
        p = s.get_state()
        s.close()
        return p
    s = state.solver
    if kind == "residual":
        th = s.theta(state.p)
        return {"theta": th, "phi": s.residual(state.x, th)}
    if kind == "rebuild":
        s.assemble(state.p)
        return {"Jx": s.apply_jacobian(state.x), "Mx": s.apply_aux(state.x), "prec": _prec(state)}
    if kind == "vcycle":
        return _prec(state)
    if kind == "gmres":
        return s.gmres(state.x)[0]
    # step: from a saved level, with the Jacobian of that level
    s.set_state(state.p)
    s.assemble(state.p)
    s.step(1)
    return s.get_state()


def _prec(state):
    """The preconditioned vector; the mixed cycle's values are single precision and are kept as such."""
    z = state.solver.apply_prec(state.x)
    return z.float() if state.c["mixed"] else z


def work(case):
    """Bytes and flops no implementation can do without: inputs read once, outputs written once; per solver
    iteration the matrix (7 FP64 coefficients), one vector in and one out, and the cycle's own data once."""
    c = case
    n = c["nx"] * c["ny"] * c["nz"]
    t = 4 if c["mixed"] else 8
    vcycle = n * (8 + 5 * t + t) * 1.25   # b, M and its diagonal, x; a quarter more for the coarse levels
    flops_v = n * 60.0
    it = n * (56 + 16) + vcycle
    kind = c["kind"]
    if kind == "residual":
        return {"bytes": n * (16.0 + 32.0), "flops": n * 300.0}
    if kind == "rebuild":
        return {"bytes": n * (16.0 + 56 + 40 + (20 if c["mixed"] else 0) + 56 + 16 + 32 + 16) + vcycle,
                "flops": n * 500.0 + flops_v}
    if kind == "vcycle":
        return {"bytes": vcycle, "flops": flops_v}
    if kind == "gmres":
        return {"bytes": 20 * it, "flops": 20 * (flops_v + 14.0 * n)}
    # Newton corrections per step and iterations per correction on these soils, at least
    if kind == "serve":
        m = sum(int(round(c["nx"] * f)) * int(round(c["ny"] * f)) * int(round(c["nz"] * f))
                for f in ((0.75, 1.0, 1.25)[r % 3] for r in range(c["requests"])))
        k = c["steps"] * 5 * 15 * m / n
    else:
        k = c["steps"] * 5 * 15
    return {"bytes": k * it, "flops": k * (flops_v + 14.0 * n)}


# ------------------------------------------------------- 64-bit reference
def _laws(p, ks):
    a = torch.where(p < 0, -p, torch.ones_like(p))
    ds = LAWS["theta_s"] - LAWS["theta_r"]
    th = LAWS["alpha"] * ds / (LAWS["alpha"] + a ** LAWS["beta"]) + LAWS["theta_r"]
    K = ks * LAWS["A"] / (LAWS["A"] + a ** LAWS["gamma"])
    return torch.where(p < 0, th, torch.full_like(p, LAWS["theta_s"])), torch.where(p < 0, K, ks + 0 * p)


def _faces(P, p, ks, axis):
    """(p_L, p_U, K_s,L, K_s,U, open) on the n+1 faces of one axis of the (z, y, x) arrays."""
    d = {0: 2, 1: 1, 2: 0}[axis]
    lo, hi = p.narrow(d, 0, 1), p.narrow(d, p.shape[d] - 1, 1)
    bl = torch.full_like(lo, P.bc_value[2 * axis])
    bu = torch.full_like(hi, P.bc_value[2 * axis + 1])
    if axis == 2 and P.patch_face == 5:
        u = (torch.arange(P.nx, device=p.device, dtype=p.dtype) + 1) * P.hx
        v = (torch.arange(P.ny, device=p.device, dtype=p.dtype) + 1) * P.hy
        inside = ((v >= P.patch_lo[1]) & (v <= P.patch_hi[1]))[:, None] & ((u >= P.patch_lo[0]) & (u <= P.patch_hi[0]))
        bu = torch.where(inside[None], torch.full_like(bu, P.patch_value), bu)
    kl, kh = ks.narrow(d, 0, 1), ks.narrow(d, ks.shape[d] - 1, 1)
    open_ = torch.ones(p.shape[d] + 1, device=p.device, dtype=p.dtype)
    open_[0], open_[-1] = float(P.bc_type[2 * axis]), float(P.bc_type[2 * axis + 1])
    shape = [1, 1, 1]
    shape[d] = -1
    return (torch.cat([bl, p], d), torch.cat([p, bu], d), torch.cat([kl, ks], d), torch.cat([ks, kh], d),
            open_.reshape(shape), d)


def _mean(P, pL, pU, KL, KU):
    if P.mean == 0:
        return 0.5 * (KL + KU)
    if P.mean == 2:
        return 2 * KL * KU / (KL + KU)
    return torch.where(pU - pL >= 0, KU, KL)


def _phi(P, ks, p, th_old):
    shape = (P.nz, P.ny, P.nx)
    p, ks = p.reshape(shape), ks.reshape(shape)
    acc = (_laws(p, ks)[0] - th_old.reshape(shape)) / P.dt
    for axis, h in enumerate((P.hx, P.hy, P.hz)):
        pL, pU, ksL, ksU, open_, d = _faces(P, p, ks, axis)
        KL, KU = _laws(pL, ksL)[1], _laws(pU, ksU)[1]
        g = _mean(P, pL, pU, KL, KU) * (pU - pL) / (h * h)
        if axis == 2:
            g = g + (KL + KU) / (2 * h)
        g = g * open_
        acc = acc - (g.narrow(d, 1, p.shape[d]) - g.narrow(d, 0, p.shape[d]))
    return acc.reshape(-1)


def _jvp(P, ks, p, x):
    th = torch.zeros_like(p)
    return torch.func.jvp(lambda q: _phi(P, ks, q, th), (p,), (x,))[1]


def _mx(P, ks, p, x):
    """The symmetric auxiliary matrix times x: frozen conductivities plus theta'/dt."""
    shape = (P.nz, P.ny, P.nx)
    dth = torch.func.jvp(lambda q: _laws(q, ks)[0], (p,), (torch.ones_like(p),))[1]
    p, ks, v = p.reshape(shape), ks.reshape(shape), x.reshape(shape)
    acc = dth.reshape(shape) / P.dt * v
    for axis, h in enumerate((P.hx, P.hy, P.hz)):
        pL, pU, ksL, ksU, open_, d = _faces(P, p, ks, axis)
        Kf = _mean(P, pL, pU, _laws(pL, ksL)[1], _laws(pU, ksU)[1]) * open_ / (h * h)
        zero = torch.zeros_like(v.narrow(d, 0, 1))
        g = Kf * (torch.cat([v, zero], d) - torch.cat([zero, v], d))
        acc = acc - (g.narrow(d, 1, v.shape[d]) - g.narrow(d, 0, v.shape[d]))
    return acc.reshape(-1)


def _dense_jacobian(P, ks, p):
    """The 7-point Jacobian as a dense matrix from 7 directional derivatives ((i + 2j + 3k) mod 7 probes)."""
    n = p.numel()
    c = torch.arange(n, device=p.device)
    i, j, k = c % P.nx, (c // P.nx) % P.ny, c // (P.nx * P.ny)
    J = torch.zeros((n, n), dtype=p.dtype, device=p.device)
    for col in range(7):
        y = _jvp(P, ks, p, ((i + 2 * j + 3 * k) % 7 == col).to(p.dtype))
        for di, dj, dk in ((0, 0, 0), (-1, 0, 0), (1, 0, 0), (0, -1, 0), (0, 1, 0), (0, 0, -1), (0, 0, 1)):
            ii, jj, kk = i + di, j + dj, k + dk
            m = ((ii >= 0) & (ii < P.nx) & (jj >= 0) & (jj < P.ny) & (kk >= 0) & (kk < P.nz)
                 & ((ii + 2 * jj + 3 * kk) % 7 == col))
            J[c[m], (ii + P.nx * (jj + P.ny * kk))[m]] = y[m]
    return J


def _newton(P, ks, p):
    """One backward-Euler step to rounding: dense Newton with step halving."""
    th = _laws(p, ks)[0]
    u = p.clone()
    for _ in range(60):
        F = _phi(P, ks, u, th)
        f = float(F.norm())
        if float(F.abs().max()) < 1e-13:
            break
        d = torch.linalg.solve(_dense_jacobian(P, ks, u), -F)
        lam = 1.0
        while lam > 1e-3 and not float(_phi(P, ks, u + lam * d, th).norm()) < f:
            lam *= 0.5
        if lam <= 1e-3:
            break
        u = u + lam * d
    return u


def exact(case, seed):
    c = case
    small = c["nx"] * c["ny"] * c["nz"] <= 4096
    if c["kind"] == "serve":
        return None
    if c["kind"] in ("gmres", "step", "simulate") and not small or c["kind"] == "vcycle":
        return None  # a large solve, or an AMG hierarchy, is out of a plain reference's reach
    P, O, ks, p, x = _inputs(c, seed)
    if c["kind"] == "residual":
        th = _laws(p, ks)[0]
        return {"theta": th, "phi": _phi(P, ks, p + 0.5 * x, th)}
    if c["kind"] == "rebuild":
        return {"Jx": _jvp(P, ks, p, x), "Mx": _mx(P, ks, p, x), "prec": None}
    p0 = torch.full_like(p, P_INIT)
    if c["kind"] == "gmres":
        b = -_phi(P, ks, p0, _laws(p0, ks)[0]) * (1.0 + 0.1 * x)
        return torch.linalg.solve(_dense_jacobian(P, ks, p0), b)
    for _ in range(2 if c["kind"] == "step" else c["steps"]):
        p0 = _newton(P, ks, p0)
    return p0
