"""The work that programs have this framework do, as cases that can be timed and compared.

A case is a dict of plain values: a grid, the physics, the storage form and one call of
the public interface (``rossbi.Sim``): ``step`` advances a simulation by some Courant
steps, ``adjoint`` records a run of steps and takes the gradient of the dust mass held by
the vortex core.  ``listed`` gives the named cases, ``draw`` more of the same ranges,
``prepare`` a simulation in mid-run, ``run`` one pass, ``work`` what a pass cannot do
without, and ``exact`` the same outputs from the plain float64 torch form of the scheme
at the end of this file.

Every simulation starts from the disc's (or the Sod annulus's) initial state with waves
in the gas and in every dust fluid and with little dust, stirred up to the gas's scale
height; it is handed over as a restart from stored fields.  The waves stand for the
turbulence of a run under way, and they matter to a comparison: undisturbed dust settles
on the midplane face with mirror symmetry, where the pressureless Riemann problem jumps
with the last bit of the state.  The small dust mass lets a coarse disc run on for the
thousands of steps that timing takes: a heavy layer falling out of the thin gas above
seven scale heights ends it within a sound crossing.
"""
import math

import numpy as np
import torch

from paper_2207_04252_amd import rossbi, synth

R_IN = 0.5  # inner radius of the disc workloads


def _case(name, nr, nth, nz, dust=0, form="fp64", call="step", steps=1, physics="base", kind="disc"):
    return {"name": name, "kind": kind, "nr": nr, "nth": nth, "nz": nz, "dust": dust, "form": form,
            "call": call, "steps": steps, "physics": physics}


def listed():
    return [
        # the smallest call: one step of the shock-tube annulus, all launches and waits
        _case("sod_annulus_1step", 256, 64, 1, kind="sod"),
        # a two-dimensional disc driven in blocks of steps, as parameter studies run it
        _case("gas_2d_50steps", 128, 256, 1, steps=50),
        # a coarse bi-fluid slice watched step by step (a grid of the tests)
        _case("bifluid_slice_1step", 24, 64, 32, dust=1),
        # the gas disc in both storage forms
        _case("gas_disc_fp64", 128, 256, 64, steps=10),
        _case("gas_disc_fp32p", 128, 256, 64, steps=10, form="fp32p"),
        # the bi-fluid disc in both storage forms
        _case("bifluid_fp64", 256, 512, 64, dust=1, steps=5),
        _case("bifluid_fp32p", 256, 512, 64, dust=1, steps=5, form="fp32p"),
        # three species on a grid that fills no tile evenly
        _case("bifluid3_ragged", 131, 197, 33, dust=3, steps=5),
        # the largest workload: three species at full resolution
        _case("bifluid3_large_fp32p", 512, 1024, 128, dust=3, steps=2, form="fp32p"),
        # every optional term of the explicit step at once: indirect gravity, the Epstein /
        # Stokes drag law, wave-killing radial and damped vertical zones
        _case("bifluid_full_physics", 256, 512, 64, dust=1, steps=5, physics="full"),
        # grains well below the step's stopping time: the split exact drag
        _case("exact_drag", 128, 256, 64, dust=1, steps=5, physics="exact_drag"),
        # gradient of the vortex-core dust mass through twenty recorded steps
        _case("adjoint_20steps", 128, 256, 32, dust=1, call="adjoint", steps=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = "adjoint" if rng.random() < 0.2 else "step"
    nr, nth = _log_int(rng, 16, 512), _log_int(rng, 16, 1024)
    nz = 1 if rng.random() < 0.15 else _log_int(rng, 24, 128)
    physics, form = "base", "fp64"
    if call == "step":
        physics = rng.choice(["base", "base", "base", "full", "outflow", "exact_drag"])
        form = rng.choice(["fp64", "fp32p"])
        cells = 3.2e7
    else:
        cells = 1.0e6
    while nr * nth * nz > cells:
        nr, nth = max(16, nr * 3 // 4), max(16, nth * 3 // 4)
    dust = rng.choice([0, 1, 3])
    # explicit drag needs steps below the smallest stopping time (Stokes number 0.01 in the
    # three-species disc): about a third of the smallest cell side at the inner edge
    side = min(R_IN * (4.0 ** (1.0 / nr) - 1.0), 2.0 * math.pi * R_IN / nth,
               0.3 / nz if nz > 1 else 1.0)
    if physics == "exact_drag" or call == "adjoint" or (dust == 3 and side / 3.0 > 0.0028):
        dust = 1
    if physics == "full" and dust == 0:
        dust = 1
    most = 2 * 512 * 1024 * 128 * 4 // (nr * nth * nz * (1 + dust))
    steps = min(_log_int(rng, 1, 20), max(1, most // (8 if call == "adjoint" else 1)))
    case = _case("", nr, nth, nz, dust, form, call, steps, physics)
    del case["name"]
    return case


def _config(case):
    """The workload of a case: the repository's own disc with that many species, rescaled."""
    if case["kind"] == "sod":
        return synth.C1_SOD.scaled(case["nr"], case["nth"], case["nz"])
    base = {0: synth.C2_DISC, 1: synth.C3_BIFLUID, 3: synth.C4_LARGE}[case["dust"]]
    if case["call"] == "adjoint":
        base = synth.C5_ADJOINT
    cfg = base.scaled(case["nr"], case["nth"], case["nz"]).with_(
        hd_over_h=(1.0,) * base.n_dust, eps_dust=(1e-4,) * base.n_dust)
    if case["physics"] == "full":
        cfg = synth.epstein_grains(cfg).with_(indirect=True, bc_r=1, bc_z=2)
    elif case["physics"] == "outflow":
        cfg = cfg.with_(bc_z=1)
    elif case["physics"] == "exact_drag":
        cfg = cfg.with_(stokes=(0.0015,), drag_exact=True)
    return cfg


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _objective(cfg, ref):
    """dJ/dE of the dust mass in the vortex core."""
    lam = torch.zeros((cfg.n_fields, cfg.nz, cfg.nr, cfg.nth), dtype=torch.float64, device=ref.dev)
    core = ((ref.rc >= synth.CORE_R[0]) & (ref.rc <= synth.CORE_R[1]))[:, None] & \
           ((ref.th - cfg.vortex_th0).abs() < synth.CORE_DTH)[None, :]
    lam[8] = ref.V[:, None] * core
    return lam


def prepare(case, seed):
    cfg = _config(case)
    ref = Reference(cfg, _device())
    sim = rossbi.Sim(cfg, precision=rossbi.RB_FP32_PERT if case["form"] == "fp32p" else rossbi.RB_FP64)
    sim.set_fields(ref.initial(seed).cpu().numpy())
    lam = _objective(cfg, ref) if case["call"] == "adjoint" else None
    return {"case": case, "cfg": cfg, "sim": sim, "lam": lam, "state": _state_views(cfg, sim, case["form"])}


def _state_views(cfg, sim, form):
    """The simulation's state buffer by the layout of the C interface."""
    shape, nd, n = (cfg.nz, cfg.nr, cfg.nth), cfg.n_dust, cfg.n_cells
    if form == "fp64":
        full = sim.state.view(torch.float64).view(5 + 4 * nd, *shape)
        return {"gas": full[:5], "dust": full[5:]} if nd else {"gas": full}
    nf32 = 5 + 3 * nd
    low = sim.state[:4 * nf32 * n].view(torch.float32).view(nf32, *shape)
    if not nd:
        return {"gas": low}
    head = (nf32 * n + 63) // 64 * 64 * 4
    dens = sim.state[head:head + 8 * nd * n].view(torch.float64).view(nd, *shape)
    return {"gas": low[:5], "dust_velocity": low[5:], "dust_density": dens}


def run(state):
    case, sim = state["case"], state["sim"]
    if case["call"] == "step":
        _, dts = sim.step(case["steps"], check=True)
        return {"dt": dts, **state["state"]}
    dts = sim.record(case["steps"], 20)
    grad, stokes = sim.adjoint(state["lam"])
    return {"dt": dts, "gradient": grad, "stokes_gradient": stokes, **state["state"]}


def work(case):
    """Per step, the stored state read once and written once, and the scheme's own
    operations of two stages (about 340 per cell for a gas face direction, 180 for a dust
    one); a gradient also reads the state and reads and writes the cotangent, and costs at
    least two operators' worth of operations again."""
    cells = case["nr"] * case["nth"] * case["nz"]
    stored = (20 + 20 * case["dust"]) if case["form"] == "fp32p" else (40 + 32 * case["dust"])
    dirs = 2 if case["nz"] == 1 else 3
    ops = 2 * dirs * (340 + 180 * case["dust"])
    adjoint = case["call"] == "adjoint"
    return {"bytes": case["steps"] * cells * stored * (5 if adjoint else 2),
            "flops": case["steps"] * cells * ops * (3 if adjoint else 1)}


def exact(case, seed):
    cfg = _config(case)
    ref = Reference(cfg, _device())
    with torch.no_grad():
        E = ref.split(ref.initial(seed))
        dts, states = [], []
        for _ in range(case["steps"]):
            dts.append(ref.cfl(E))
            states.append(E if case["call"] == "adjoint" else None)
            E = ref.step(E, dts[-1])
    out = {"dt": np.array(dts)}
    if case["call"] == "adjoint":
        lam, stokes = ref.gradient(states, dts, _objective(cfg, ref))
        out.update(gradient=lam, stokes_gradient=stokes)
    if case["form"] == "fp64":
        out["gas"] = E[:5]
        if cfg.n_dust:
            out["dust"] = E[5:]
        return out
    out["gas"] = E[:5]
    if cfg.n_dust:
        dens = E[8::4]
        vel = torch.stack([E[5 + 4 * s + c] / dens[s] for s in range(cfg.n_dust) for c in range(3)])
        vel[1::3] -= ref.W0[1]
        out.update(dust_velocity=vel, dust_density=dens)
    return out


class Reference:
    """The scheme in plain float64 torch: the parabolic primitive reconstruction with its
    MinMod limiter, exact gas and pressureless Riemann fluxes, geometric, gravity, drag and
    indirect sources, damping, the balanced RK2 step and its Courant step.  States are
    (field, z, r, theta): the gas deviation from the stationary flow, then the dust fluids'
    momenta and density."""

    def __init__(self, cfg, dev):
        self.cfg, self.dev = cfg, dev
        self.g = cfg.gamma
        nr, nth, nz = cfg.nr, cfg.nth, cfg.nz
        self.twod = nz == 1
        self.disc = cfg.init_kind == synth.INIT_DISC
        dth = 2.0 * math.pi / nth
        dz = 1.0 if self.twod else 2.0 * cfg.z_half / nz
        i = torch.arange(-2, nr + 3, dtype=torch.float64, device=dev)
        if cfg.log_r:
            rf = cfg.r_in * (cfg.r_out / cfg.r_in) ** (i / nr)
        else:
            rf = cfg.r_in + i * ((cfg.r_out - cfg.r_in) / nr)
        rc = 0.5 * (rf[:-1] + rf[1:])                 # centres of cells -2 .. nr + 1
        self.rp, self.rf, self.rc = rc, rf[2:nr + 3], rc[2:nr + 2]
        k = torch.arange(-2, nz + 2, dtype=torch.float64, device=dev)
        zc = torch.zeros(5, dtype=torch.float64, device=dev) if self.twod else (k + 0.5 - 0.5 * nz) * dz
        self.zp, self.zc = zc, zc[2:nz + 2]
        self.th = (torch.arange(nth, dtype=torch.float64, device=dev) + 0.5) * dth
        rm, rq = self.rf[:-1], self.rf[1:]
        area = 0.5 * (rq * rq - rm * rm)
        self.V, self.Ar = area * dth * dz, self.rf * dth * dz
        self.Ath, self.Az = (rq - rm) * dz, area * dth
        self.maxA = torch.maximum(torch.maximum(self.Ar[:-1], self.Ar[1:]), self.Ath)
        if not self.twod:
            self.maxA = torch.maximum(self.maxA, self.Az)
        self.dz, self.dth = dz, dth
        self.omega = torch.sqrt(cfg.GM / self.rc ** 3)
        # parabola weights and limiter bounds along r of cells -1 .. nr
        hm, hp = rc[1:-1] - rc[:-2], rc[2:] - rc[1:-1]
        self.weights = []
        for d in (rf[2:-1] - rc[1:-1], rf[1:-2] - rc[1:-1]):
            wp, wm = (d * d + hm * d) / (hp * (hm + hp)), (hp * d - d * d) / (hm * (hm + hp))
            self.weights.append([x[None, :, None] for x in (wm, wp, 2.0 * d / hm, 2.0 * d / hp)])
        col = self.rc[None, :, None]
        s3 = (col ** 2 + self.zc[:, None, None] ** 2) ** 1.5
        self.gr, self.gz = -cfg.GM * col / s3, -cfg.GM * self.zc[:, None, None] / s3
        self.W0 = self.background(self.rc, self.zc)   # stationary primitives (u, v, w, p, rho)
        self.E0 = self.conserved(self.W0)
        self.W0r = self.background(self.rf, self.zc)
        if not self.twod:
            zf = (torch.arange(nz + 1, dtype=torch.float64, device=dev) - 0.5 * nz) * dz
            self.W0z = self.background(self.rc, zf)
        self.inv_st = [torch.tensor(1.0 / s, dtype=torch.float64, device=dev) for s in cfg.stokes]
        self.damping = self._damping()
        self._R0 = None

    # ---- the stationary flow, the initial state

    def background(self, r, z):
        """Stationary primitives at radii r and heights z, shape (5, z, r, 1); zero for the annulus."""
        c = self.cfg
        shape = (z.numel(), r.numel(), 1)
        if not self.disc:
            return torch.zeros((5,) + shape, dtype=torch.float64, device=self.dev)
        r, z = r[None, :, None], z[:, None, None]
        c2 = c.h0 ** 2 * c.GM * r ** c.beta_T
        s = torch.sqrt(r * r + z * z)
        rho = c.rho_mid0 * r ** c.beta_rho * torch.exp(c.GM / c2 * (1.0 / s - 1.0 / r))
        v = torch.sqrt(c.GM / r + c2 * (c.beta_T + c.beta_rho) + c.beta_T * c.GM * (1.0 / r - 1.0 / s))
        zero = torch.zeros(shape, dtype=torch.float64, device=self.dev)
        return torch.stack([zero, v, zero, c2 * rho, rho])

    def thickness(self, hd_over_h, r):
        """Scale height of a layer at radii r, from its ratio to the gas's."""
        c = self.cfg
        return hd_over_h * torch.sqrt(c.h0 ** 2 * c.GM * r ** c.beta_T) / torch.sqrt(c.GM / r ** 3)

    def layer(self, s, r, z):
        """Initial dust density of species s."""
        c = self.cfg
        r, z = r[None, :, None], z[:, None, None]
        hd = self.thickness(c.hd_over_h[s], r)
        return (c.eps_dust[s] / c.hd_over_h[s] * c.rho_mid0 * r ** c.beta_rho
                * torch.exp(-z * z / (2.0 * hd * hd)))

    def conserved(self, W):
        u, v, w, p, rho = W
        return torch.stack([rho * u, rho * v, rho * w,
                            p / (self.g - 1.0) + 0.5 * rho * (u * u + v * v + w * w), rho])

    def initial(self, seed):
        """The full fields of a run under way: the stationary flow with a weak pressure bump
        in radial balance (temperature kept), vortex, density noise, waves."""
        c = self.cfg
        shape = (c.nz, c.nr, c.nth)
        rng = torch.Generator(device=self.dev).manual_seed(int(seed))
        few = torch.Generator().manual_seed(int(seed) + 1)

        def noise():
            return 2.0 * torch.rand(shape, dtype=torch.float64, device=self.dev, generator=rng) - 1.0

        def waves():
            """Four smooth modes of random wavenumbers and phases, of unit amplitude."""
            x = torch.log(self.rc / self.rc[0])[None, :, None]
            z = (self.zc / c.z_half)[:, None, None]
            out = torch.zeros(shape, dtype=torch.float64, device=self.dev)
            for _ in range(4):
                a = torch.rand(4, generator=few, dtype=torch.float64).tolist()
                out += 0.25 * torch.cos(int(1 + 6 * a[0]) * self.th + 20.0 * (a[1] - 0.5) * x
                                        + 4.0 * (a[2] - 0.5) * z + 2.0 * math.pi * a[3])
            return out

        if not self.disc:
            left = (self.rc < c.sod_r0)[None, :, None]
            rho, p, u = (torch.where(left, a, b) * torch.ones(shape, dtype=torch.float64, device=self.dev)
                         for a, b in zip(torch.tensor(c.sod_left, device=self.dev, dtype=torch.float64),
                                         torch.tensor(c.sod_right, device=self.dev, dtype=torch.float64)))
            zero = torch.zeros_like(rho)
            return self.conserved([u, zero, zero, p, rho * (1.0 + 1e-3 * noise())])
        X = self.rc[None, :, None] - c.vortex_r0
        Y = c.vortex_r0 * (self.th - c.vortex_th0)[None, None, :]
        a, b = c.vortex_sig_r ** -2, c.vortex_sig_a ** -2
        psi = (-2.0 * math.sqrt(c.GM / c.vortex_r0 ** 3) / (a + b)
               * torch.exp(-0.5 * X * X * a - 0.5 * Y * Y * b))
        # the waves are weak and stay inside the layer: rising into thin gas they steepen as
        # the inverse root of its density, and a grain up there falls in less than a step
        col = (self.zc[:, None, None] / self.thickness(1.0, self.rc)[None, :, None]) ** 2
        stir = 2e-4 * c.h0 * torch.exp(-col)          # velocity, in units of r Omega
        u = c.vortex_amp * (-psi * c.vortex_r0 * Y * b / self.rc[None, :, None])
        gauss = torch.exp(-0.5 * X * X / 0.05 ** 2)
        bump = 1.0 + 0.01 * gauss
        c2 = self.W0[3] / self.W0[4]
        v = torch.sqrt(self.W0[1] ** 2 - self.rc[None, :, None] * c2 * 0.01 * gauss * X / 0.05 ** 2 / bump)
        v = v + c.vortex_amp * psi * X * a
        rho = self.W0[4] * bump * (1.0 + c.noise_amp * noise())
        p = self.W0[3] * bump * (1.0 + stir * waves())
        fields = list(self.conserved([u + stir * waves(), v + stir * waves(), stir * waves(), p, rho]))
        for s in range(c.n_dust):
            rd = self.layer(s, self.rc, self.zc) * (1.0 + c.noise_amp * noise())
            fields += [rd * (u + stir * waves()), rd * (v + stir * waves()), rd * stir * waves(), rd]
        return torch.stack(fields)

    def split(self, full):
        """Full fields -> the stored state (the gas as a deviation)."""
        if self.disc:
            full = full.clone()
            full[:5] -= self.E0
        return full

    # ---- the operator

    def primitives(self, E):
        """Gas primitives (u, v, w, p, rho) of a stored state."""
        q = E[:5] + self.E0 if self.disc else E[:5]
        u, v, w = q[0] / q[4], q[1] / q[4], q[2] / q[4]
        return torch.stack([u, v, w, (self.g - 1.0) * (q[3] - 0.5 * (q[0] * u + q[1] * v + q[2] * w)), q[4]])

    def _ghosts(self, X, axis, lo, hi):
        """X with two cells lo and hi before and after it along axis (1 z, 2 r)."""
        shape = list(X.shape)
        shape[axis] = 2
        return torch.cat([lo.expand(shape), X, hi.expand(shape)], axis)

    def _ghost_cells(self, X, axis, species):
        """The two cells beyond each end along an axis: the stationary flow, or the outflow copy."""
        n = X.shape[axis]
        if axis == 1 and self.cfg.bc_z == 1:
            if species is not None:
                return X[:, :1], X[:, -1:]
            # the boundary cell's gas deviation scaled by the stationary densities' ratio
            sides = []
            for edge, z in ((0, self.zp[:2]), (n - 1, self.zp[-2:])):
                base = self.W0[:, edge:edge + 1]
                scale = self.background(self.rc, z)[4] / base[4]
                ghost = self.background(self.rc, z)
                dev = (self.conserved(base + X[:, edge:edge + 1]) - self.conserved(base)) * scale
                q = self.conserved(ghost) + dev
                u, v, w = q[0] / q[4], q[1] / q[4], q[2] / q[4]
                P = (self.g - 1.0) * (q[3] - 0.5 * (q[0] * u + q[1] * v + q[2] * w))
                sides.append(torch.stack([u, v, w, P, q[4]]) - ghost)
            return sides
        if species is None:
            zero = torch.zeros((5, 1, 1, 1), dtype=torch.float64, device=self.dev)
            if self.disc:
                return zero, zero
            inner, outer = X.new_tensor(self.cfg.sod_left), X.new_tensor(self.cfg.sod_right)
            return tuple(torch.stack([s[2], s[0] * 0, s[0] * 0, s[1], s[0]]).reshape(5, 1, 1, 1)
                         for s in (inner, outer))
        sides = []
        for e in (slice(0, 2), slice(-2, None)):
            r, z = (self.rp[e], self.zc) if axis == 2 else (self.rc, self.zp[e])
            W = self.background(r, z)
            sides.append(torch.stack([W[0], W[1], W[2], self.layer(species, r, z)]))
        return sides

    @staticmethod
    def _minmod(x, y, z):
        lo, hi = torch.minimum(x, torch.minimum(y, z)), torch.maximum(x, torch.maximum(y, z))
        return torch.where(lo > 0.0, lo, torch.where(hi < 0.0, hi, torch.zeros_like(x)))

    def _faces(self, X, axis, species=None):
        """Limited face states (left, right) and the two cells' own values at every face
        along an axis (1 z, 2 r, 3 theta): faces 0 .. n, or for theta the upper face of
        each cell."""
        if axis == 3:
            A, B, C, D = torch.roll(X, 1, 3), X, torch.roll(X, -1, 3), torch.roll(X, -2, 3)
        else:
            P = self._ghosts(X, axis, *self._ghost_cells(X, axis, species))
            n = X.shape[axis] + 1
            A, B, C, D = (P.narrow(axis, o, n) for o in range(4))
        d1, d2, d3 = B - A, C - B, D - C
        if axis == 2:
            n = X.shape[2] + 1
            wm, wp, lm, lp = (x[:, :n] for x in self.weights[0])
            up = self._minmod(wp * d2 + wm * d1, lm * d1, lp * d2)
            wm, wp, lm, lp = (x[:, 1:n + 1] for x in self.weights[1])
            lo = self._minmod(wp * d3 + wm * d2, lm * d2, lp * d3)
        else:
            up = self._minmod((3.0 * d2 + d1) / 8.0, d1, d2)
            lo = self._minmod(-(3.0 * d2 + d3) / 8.0, -d2, -d3)
        return B + up, C + lo, B, C

    def _pressure(self, p, rK, pK, cK):
        """Pressure function of one side of the gas Riemann problem, and its slope."""
        g = self.g
        A, B = 2.0 / ((g + 1.0) * rK), (g - 1.0) / (g + 1.0) * pK
        q = torch.sqrt(A / (p + B))
        x = (p / pK) ** ((g - 1.0) / (2.0 * g))
        shock = p > pK
        f = torch.where(shock, (p - pK) * q, 2.0 * cK / (g - 1.0) * (x - 1.0))
        return f, torch.where(shock, q * (1.0 - 0.5 * (p - pK) / (p + B)), x * pK / (p * rK * cK))

    def _gas_flux(self, L, R, n):
        """Flux of the exact Riemann solution at x/t = 0 between primitive states along
        velocity component n (no vacuum: these flows make none)."""
        g = self.g
        cL, cR = torch.sqrt(g * L[3] / L[4]), torch.sqrt(g * R[3] / R[4])
        du = R[n] - L[n]
        with torch.no_grad():
            p = 0.5 * (L[3] + R[3]) - 0.125 * du * (L[4] + R[4]) * (cL + cR)
            p = torch.maximum(p, 1e-8 * torch.minimum(L[3], R[3]))
            for _ in range(30):
                fL, dL = self._pressure(p, L[4], L[3], cL)
                fR, dR = self._pressure(p, R[4], R[3], cR)
                new = torch.maximum(p - (fL + fR + du) / (dL + dR), 1e-8 * p)
                done = bool(((new - p).abs() <= 1e-13 * new).all())
                p = new
                if done:
                    break
            slope = self._pressure(p, L[4], L[3], cL)[1] + self._pressure(p, R[4], R[3], cR)[1]
        # one differentiable Newton step carries the derivative of the star pressure
        fL, fR = self._pressure(p, L[4], L[3], cL)[0], self._pressure(p, R[4], R[3], cR)[0]
        p = p - (fL + fR + du) / slope
        us = 0.5 * (L[n] + R[n]) + 0.5 * (self._pressure(p, R[4], R[3], cR)[0]
                                          - self._pressure(p, L[4], L[3], cL)[0])
        left = us >= 0.0
        # mirrored to the left side: K the side of the contact, uK towards the contact
        K = torch.where(left, L, R)
        sg = torch.where(left, 1.0, -1.0)
        cK, uK, u = torch.where(left, cL, cR), sg * K[n], sg * us
        x = p / K[3]
        k = (g - 1.0) / (g + 1.0)
        shock = x > 1.0
        speed = uK - cK * torch.sqrt((g + 1.0) / (2.0 * g) * x + (g - 1.0) / (2.0 * g))
        rare = x ** ((g - 1.0) / (2.0 * g))
        outer = torch.where(shock, speed >= 0.0, uK - cK >= 0.0)
        fan = ~shock & ~outer & (u - cK * rare >= 0.0)
        cc = 2.0 / (g + 1.0) * (cK + 0.5 * (g - 1.0) * uK)
        ratio = torch.where(fan, cc / cK, torch.ones_like(cc))
        rho = torch.where(shock, K[4] * (x + k) / (k * x + 1.0), K[4] * x ** (1.0 / g))
        rho = torch.where(fan, K[4] * ratio ** (2.0 / (g - 1.0)), rho)
        rho = torch.where(outer, K[4], rho)
        P = torch.where(outer, K[3], torch.where(fan, K[3] * ratio ** (2.0 * g / (g - 1.0)), p))
        un = torch.where(outer, K[n], torch.where(fan, sg * cc, us))
        W = [un if c == n else K[c] for c in range(3)]
        m = rho * un
        F = [m * W[c] + (P if c == n else 0.0) for c in range(3)]
        en = P / (g - 1.0) + 0.5 * rho * (W[0] ** 2 + W[1] ** 2 + W[2] ** 2)
        return torch.stack(F + [(en + P) * un, m])

    @staticmethod
    def _dust_flux(L, R, n):
        """Flux of the pressureless Riemann solution: the upwind state, nothing between
        diverging streams, the delta shock's side between converging ones."""
        meet = L[n] > R[n]
        num = torch.sqrt(L[3]) * L[n] + torch.sqrt(R[3]) * R[n]
        wl = torch.where(meet, (num > 0.0).double() + 0.5 * (num == 0.0).double(), (L[n] > 0.0).double())
        wr = torch.where(meet, (num < 0.0).double() + 0.5 * (num == 0.0).double(),
                         ((R[n] < 0.0) & ~(L[n] > 0.0)).double())
        fl = torch.stack([L[3] * L[n] * L[0], L[3] * L[n] * L[1], L[3] * L[n] * L[2], L[3] * L[n]])
        fr = torch.stack([R[3] * R[n] * R[0], R[3] * R[n] * R[1], R[3] * R[n] * R[2], R[3] * R[n]])
        return wl * fl + wr * fr

    def _divergence(self, X, species=None):
        """-sum over faces of area times flux, of the reconstructed variables X."""
        total = 0.0
        for axis, n, area in ((2, 0, None), (3, 1, self.Ath), (1, 2, self.Az)):
            if axis == 1 and self.twod:
                continue
            L, R, B, C = self._faces(X, axis, species)
            if species is None:
                face = self.W0r if axis == 2 else (self.W0 if axis == 3 else self.W0z)
                cell = self._centres(axis)
                L, R = L + face, R + face
                L = torch.where((L[3] > 0.0) & (L[4] > 0.0), L, B + cell[0])
                R = torch.where((R[3] > 0.0) & (R[4] > 0.0), R, C + cell[1])
                F = self._gas_flux(L, R, n)
            else:
                F = self._dust_flux(torch.where(L[3] < 0.0, B, L), torch.where(R[3] < 0.0, C, R), n)
            if axis == 2:
                F = F * self.Ar[None, None, :, None]
                total = total - (F[:, :, 1:] - F[:, :, :-1])
            else:
                d = F - torch.roll(F, 1, 3) if axis == 3 else F[:, 1:] - F[:, :-1]
                total = total - area[None, None, :, None] * d
            del L, R, B, C, F
        return total

    def _centres(self, axis):
        """Stationary primitives at the centres of the two cells next to each face."""
        if axis == 3:
            return self.W0, self.W0
        if axis == 2:
            W = self.background(self.rp[1:-1], self.zc)
            return W[:, :, :-1], W[:, :, 1:]
        W = self.background(self.rc, self.zp[1:-1])
        return W[:, :-1], W[:, 1:]

    def _rates(self, W, s):
        """Inverse stopping time of species s in gas W."""
        c = self.cfg
        if c.drag_law == 0:
            return self.omega[None, :, None] * self.inv_st[s]
        epstein = torch.sqrt(W[3] * W[4]) / (c.grain_density[s] * c.grain_size[s])
        x = 4.0 * c.grain_size[s] / 9.0 * W[4]
        return torch.where(x <= c.mfp_coef, epstein, epstein * c.mfp_coef / x)

    def residual(self):
        """The empty run: G of the stationary gas (axisymmetric, so of one column)."""
        if self._R0 is None:
            with torch.no_grad():
                self._R0 = self.operator(torch.zeros_like(self.W0), empty=True)
        return self._R0

    def operator(self, E, empty=False):
        """G(E) - R0; with empty, the gas alone without drag and residual (G itself)."""
        c = self.cfg
        W = self.primitives(E)
        u, v, w, p, rho = W
        ir = 1.0 / self.rc[None, :, None]
        G = self._divergence(W - self.W0)
        S = [(rho * v * v + p) * ir + rho * self.gr, -rho * u * v * ir, rho * self.gz,
             rho * (u * self.gr + w * self.gz), torch.zeros_like(rho)]
        vol = self.V[None, :, None]
        if empty:
            return G + torch.stack(S) * vol
        frame = None
        if c.indirect:
            s2 = self.rc[None, :, None] ** 2 + self.zc[:, None, None] ** 2
            mass = (rho + sum(E[8 + 4 * s] for s in range(c.n_dust))) * vol * self.rc[None, :, None] / s2 ** 1.5
            cs, sn = torch.cos(self.th), torch.sin(self.th)
            A, B = (mass * cs).sum(), (mass * sn).sum()
            frame = (-c.GM * (A * cs + B * sn), -c.GM * (B * cs - A * sn))
        dust = []
        for s in range(c.n_dust):
            m, rd = E[5 + 4 * s:8 + 4 * s], E[8 + 4 * s]
            vd = m / rd
            Gd = self._divergence(torch.cat([vd, rd[None]]), species=s)
            f = [torch.zeros_like(rd)] * 3
            if not c.drag_exact:
                its = self._rates(W, s)
                f = [rd * (vd[q] - W[q]) * its for q in range(3)]
            Sd = [rd * vd[1] ** 2 * ir + rd * self.gr - f[0], -rd * vd[0] * vd[1] * ir - f[1],
                  rd * self.gz - f[2], torch.zeros_like(rd)]
            if frame:
                Sd[0], Sd[1] = Sd[0] + rd * frame[0], Sd[1] + rd * frame[1]
            dust.append(Gd + torch.stack(Sd) * vol)
            S = [S[0] + f[0], S[1] + f[1], S[2] + f[2], S[3] + u * f[0] + v * f[1] + w * f[2], S[4]]
        if frame:
            S = [S[0] + rho * frame[0], S[1] + rho * frame[1], S[2],
                 S[3] + rho * (u * frame[0] + v * frame[1]), S[4]]
        S = torch.stack(S)
        if self.damping is not None:
            S = S - self.damping * E[:5]
        G = G + S * vol
        if c.balanced:
            G = G - self.residual()
        return torch.cat([G] + dust)

    def _damping(self):
        """Relaxation rate of the boundary zones."""
        c = self.cfg
        if c.bc_r != 1 and (c.bc_z != 2 or self.twod):
            return None
        r, z = self.rc[None, :, None], self.zc[:, None, None].abs()
        rate = torch.zeros_like(r + z)
        if c.bc_r == 1:
            for edge, wall in ((c.damp_r_in * c.r_in, c.r_in), (c.damp_r_out * c.r_out, c.r_out)):
                x = torch.clamp((r - edge) / (wall - edge), min=0.0)
                rate = rate + x * x * math.sqrt(c.GM / wall ** 3) / (2.0 * math.pi * c.damp_tau)
        if c.bc_z == 2 and not self.twod:
            x = torch.clamp((z - c.damp_z * c.z_half) / (c.z_half * (1.0 - c.damp_z)), min=0.0)
            rate = rate + x * x * self.omega[None, :, None] / (2.0 * math.pi * c.damp_tau)
        return rate

    # ---- the step

    def cfl(self, E):
        u, v, w, p, rho = self.primitives(E)
        speed = torch.sqrt(u * u + v * v + w * w) + torch.sqrt(self.g * p / rho)
        for s in range(self.cfg.n_dust):
            m, rd = E[5 + 4 * s:8 + 4 * s], E[8 + 4 * s]
            speed = torch.maximum(speed, torch.sqrt((m * m).sum(0)) / rd)
        return float((self.cfg.cfl * (self.V / self.maxA)[None, :, None] / speed).min())

    def stage(self, base, E, dt):
        return base + dt / self.V[None, None, :, None] * self.operator(E)

    def step(self, E, dt):
        if self.cfg.drag_exact:
            E = self.relax(E, 0.5 * dt)
        E = self.stage(E, self.stage(E, E, 0.5 * dt), dt)
        return self.relax(E, 0.5 * dt) if self.cfg.drag_exact else E

    def relax(self, E, tau):
        """The drag alone over tau, densities and stopping times held: the velocity
        differences decay by the matrix exponential, the total momentum stays."""
        nd = self.cfg.n_dust
        if nd == 0:
            return E
        W = self.primitives(E)
        rd = E[8::4]
        ia = torch.stack([self._rates(W, s).expand(rd[0].shape) for s in range(nd)])
        B = -(rd / W[4] * ia).movedim(0, -1)[..., None, :].expand(*rd.shape[1:], nd, nd) \
            - torch.diag_embed(ia.movedim(0, -1))
        decay = torch.linalg.matrix_exp(tau * B) if nd > 1 else torch.exp(tau * B)
        out = E.clone()
        total = W[4] + rd.sum(0)
        change = 0.0
        for c in range(3):
            ud = E[5 + c::4] / rd
            d = (decay @ (ud - W[c]).movedim(0, -1)[..., None])[..., 0].movedim(-1, 0)
            ug = (W[4] * W[c] + (rd * ud).sum(0) - (rd * d).sum(0)) / total
            change = change + 0.5 * W[4] * (ug * ug - W[c] * W[c])
            out[c] = E[c] + W[4] * (ug - W[c])
            out[5 + c::4] = rd * (ug + d)
        out[3] = E[3] + change
        return out

    def gradient(self, states, dts, lam):
        """d(lam . final state)/d(initial state) at fixed steps, and by Stokes number."""
        stokes = torch.tensor(self.cfg.stokes, dtype=torch.float64, device=self.dev, requires_grad=True)
        total = torch.zeros_like(stokes)
        kept = self.inv_st
        self.inv_st = [1.0 / stokes[s] for s in range(self.cfg.n_dust)]
        for E, dt in zip(reversed(states), reversed(dts)):
            with torch.no_grad():
                mid = self.stage(E, E, 0.5 * dt)
            x = mid.requires_grad_(True)
            self.inv_st = [1.0 / stokes[s] for s in range(self.cfg.n_dust)]
            nu, gs = torch.autograd.grad(self.operator(x), (x, stokes), dt / self.V[None, None, :, None] * lam)
            total = total + gs
            x = E.detach().requires_grad_(True)
            self.inv_st = [1.0 / stokes[s] for s in range(self.cfg.n_dust)]
            mu, gs = torch.autograd.grad(self.operator(x), (x, stokes), 0.5 * dt / self.V[None, None, :, None] * nu)
            total = total + gs
            lam = lam + nu + mu
        self.inv_st = kept
        return lam, total.detach().cpu().numpy()
