"""The framework's performance cases: what a user's program has it do.

Three groups of calls.  A simulation advances the state by full steps
(Context.step) and looks at it now and then (energy, wall fluxes and torques,
probes), restarting at another resolution from time to time.  Programs with
a time integrator of their own call the two halves, the nonlinear term and
the implicit radial stage.  Optimal-perturbation searches call the step's
vector--Jacobian product and the gradient of a rollout.  Grids run from the
small isothermal one (32 points, 16 x 31 modes) to the counter-rotating
turbulent one (128 points, 256 x 511 modes); transforms of any 5-smooth
length are allowed, so ragged grids are ordinary.

Reference values (exact) are plain FP64 numpy/torch on the host: FFTs on the
3/2-rule grid, dense solves per Fourier mode, autograd for the adjoint.
"""
import math

import numpy as np
import torch

TWO_PI = 2.0 * math.pi
C128 = torch.complex128
F64 = torch.float64


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(call, N_r, M_theta, M_z, name=None, geometry="couette", Re_i=100.0, Re_o=0.0, eta=0.71,
          Ra=0.0, precision="fp64", dynamic=False, amp=1e-3, **more):
    c = dict(call=call, geometry=geometry, N_r=N_r, M_theta=M_theta, M_z=M_z, Re_i=Re_i, Re_o=Re_o,
             eta=eta, Ra=Ra, Pr=0.7 if Ra else 1.0, precision=precision, dynamic=dynamic, amp=amp,
             L_z=2 * TWO_PI if geometry == "pipe" else TWO_PI)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # production runs: one predictor--corrector step.  The smallest grid
        # in plain FP64 at a fixed step size: many short kernels.
        _case("step", 32, 16, 31, "step-n32", Re_i=50.0, eta=0.5),
        # heated flow on 192 x 192 points, mixed precision, dynamic step size
        _case("step", 64, 64, 127, "step-heated-n64", Ra=1.0e4, precision="mixed", dynamic=True),
        # the pipe variant at the same resolution
        _case("step", 64, 64, 127, "step-pipe-n64", geometry="pipe", Re_i=4000.0, precision="mixed",
              dynamic=True, amp=1.0),
        # counter-rotating turbulence on 768 x 768 points: the largest
        _case("step", 128, 256, 511, "step-turb-n128", Re_i=2000.0, Re_o=-1000.0,
              precision="mixed", dynamic=True, amp=1e-2),
        # the nonlinear term alone (programs with their own integrator), with
        # the CFL bound: a ragged heated grid (120 x 120 points) ...
        _case("nonlinear", 49, 40, 79, "nonlinear-ragged", Ra=1.0e4),
        # ... and 384 x 384 points
        _case("nonlinear", 96, 128, 255, "nonlinear-n96"),
        # the implicit stage alone with its pressure, on a ragged heated grid
        _case("solve", 75, 48, 95, "solve-ragged", Ra=1.0e4, pressure=True),
        # the implicit stage where an adaptive integrator changes the step
        # size: the radial operators are factorised anew before each solve
        _case("solve", 64, 64, 127, "solve-new-dt", Ra=1.0e4, new_dt=True),
        # adjoint: vector--Jacobian product of one step (the stage states at
        # hand), and the gradient of the energy after a short rollout
        _case("vjp", 64, 32, 63, "vjp-n64", Re_i=200.0),
        _case("gradient", 32, 16, 31, "gradient-n32", Re_i=50.0, eta=0.5, steps=8, ckpt=4),
        # a look at the state: energy, wall fluxes and torques, probe points
        _case("monitor", 64, 64, 127, "monitor-heated", Ra=1.0e4),
        # restart of the heated run on a finer grid
        _case("remap", 96, 96, 191, "remap-n64-n96", Ra=1.0e4, from_N_r=64, from_M_theta=64,
              from_M_z=127),
    ]


# 5-smooth counts of modes (three times each is a transform length)
_SMOOTH = sorted(2 ** a * 3 ** b * 5 ** c for a in range(9) for b in range(6) for c in range(4)
                 if 4 <= 2 ** a * 3 ** b * 5 ** c <= 256)


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _modes(rng, lo, hi):
    x = _log(rng, lo, hi)
    return min(_SMOOTH, key=lambda s: abs(math.log(s / x)))


def draw(rng):
    call = rng.choice(["step"] * 5 + ["nonlinear"] * 3 + ["solve"] * 4 + ["vjp"] * 2 +
                      ["gradient", "monitor", "remap"])
    small = call in ("gradient", "remap")
    N_r = int(_log(rng, 12, 96 if small else 129))
    M_theta = _modes(rng, 5, 48 if small else 160)
    M_z = 2 * _modes(rng, max(4, M_theta // 2), min(2 * M_theta, 48 if small else 192)) - 1
    kw = {}
    if rng.random() < 0.45:
        kw["Ra"] = 1.0e4
    if call in ("step", "nonlinear", "solve") and rng.random() < 0.2:
        kw = dict(geometry="pipe", Re_i=2000.0, amp=0.5)
    if call == "step":
        kw["precision"] = rng.choice(["mixed", "fp64"])
        kw["dynamic"] = rng.random() < 0.7
    elif call == "solve":
        kw["pressure"] = rng.random() < 0.5
        kw["new_dt"] = rng.random() < 0.25
    elif call == "gradient":
        kw["steps"] = rng.randint(3, 8)
        kw["ckpt"] = rng.randint(2, 4)
    elif call == "remap":
        kw["from_N_r"] = int(_log(rng, 12, 96))
        kw["from_M_theta"] = _modes(rng, 5, 64)
        kw["from_M_z"] = 2 * _modes(rng, 5, 48) - 1
    return _case(call, N_r, M_theta, M_z, **kw)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Geo:
    """Plain data of a case: grid, base flow, derivative matrices."""

    def __init__(self, c, N_r=None, M_theta=None, M_z=None):
        self.pipe = c["geometry"] == "pipe"
        self.n = N_r or c["N_r"]
        self.Mt = M_theta or c["M_theta"]
        self.Mz = M_z or c["M_z"]
        self.K = (self.Mz - 1) // 2
        self.Nt, self.Nz = 3 * self.Mt, 3 * (self.K + 1)
        self.Lz = c["L_z"]
        self.kz = TWO_PI / self.Lz
        self.Re_i, self.Re_o, self.Ra, self.Pr = c["Re_i"], c["Re_o"], c["Ra"], c["Pr"]
        self.heated = bool(self.Ra)
        self.F = 4 if self.heated else 3
        n = self.n
        j = np.arange(n, dtype=np.longdouble)
        pi = np.longdouble("3.14159265358979323846264338327950288")
        if self.pipe:
            self.ri, self.ro, self.A, self.B = 0.0, 1.0, 0.0, 0.0
            self.r = np.cos(pi * (n - 1 - j) / (2 * n - 1)).astype(np.float64)
        else:
            eta = c["eta"]
            self.eta = eta
            self.ri, self.ro = eta / (1 - eta), 1 / (1 - eta)
            self.A = (self.Re_o * self.ro - self.Re_i * self.ri) / (self.ro ** 2 - self.ri ** 2)
            self.B = self.ri * (self.Re_i - self.A * self.ri)
            self.r = (0.5 * (self.ri + self.ro) + 0.5 * np.cos(pi * (n - 1 - j) / (n - 1))).astype(
                np.float64)

    def shape(self):
        return (self.F, self.n, self.Mt, self.Mz)

    def dt(self):
        """A step size just inside the CFL bound 0.5 of the basic flow."""
        if self.pipe:
            return 0.45 * self.Lz / self.Nz / self.Re_i
        speed = [(self.ri, abs(self.Re_i)), (self.ro, abs(self.Re_o))]
        return min([1e-3] + [0.45 * r * TWO_PI / self.Nt / s for r, s in speed if s])


def _amplitudes(g, F, seed, dev):
    """Complex normal amplitudes decaying as exp(-|(m, k)| / 4), m = 0 Hermitian."""
    gen = np.random.Generator(np.random.PCG64(seed))
    a = torch.from_numpy(gen.standard_normal((F, g.Mt, g.Mz, 2))).to(dev)
    a = torch.view_as_complex(a) * math.sqrt(0.5)
    m = torch.arange(g.Mt, dtype=F64, device=dev)[:, None]
    k = torch.arange(g.Mz, dtype=F64, device=dev)[None, :] - g.K
    a = a * torch.exp(-torch.sqrt(m * m + k * k) / 4)
    a[:, 0] = 0.5 * (a[:, 0] + torch.flip(a[:, 0], (-1,)).conj())
    a[:, 0, g.K] = a[:, 0, g.K].real.to(C128)
    return a


def _field(g, seed, dev, scale=1.0, walls=True, F=None):
    """Smooth random fields [F][N_r][M_theta][M_z]; walls: zero at the walls
    (pipe: regular at the axis)."""
    F = F or g.F
    a = _amplitudes(g, 2 * F, seed, dev) * scale
    r = torch.from_numpy(g.r).to(dev)[:, None, None]
    if g.pipe:
        def prof(q):
            peak = (q / (q + 4.0)) ** (q / 2.0) * (4.0 / (q + 4.0)) ** 2
            return r ** q * (1 - r * r) ** 2 / peak
        m = torch.arange(g.Mt, dtype=F64, device=dev)[None, :, None]
        up = (a[0] + 1j * a[1]) * prof(m + 1)
        um = (a[0] - 1j * a[1]) * prof((m - 1).abs())
        return torch.stack([0.5 * (up + um), -0.5j * (up - um), a[2] * prof(m)]).contiguous()
    x = 2 * (r - g.ri) / (g.ro - g.ri) - 1
    w = (1 - x * x) ** 2 if walls else torch.ones_like(x)
    out = torch.empty((F, g.n, g.Mt, g.Mz), dtype=C128, device=dev)
    for f in range(F):
        out[f] = w * (a[f] + a[F + f] * x)
    return out


def _base(g, dev):
    u = torch.zeros(g.shape(), dtype=C128, device=dev)
    r = torch.from_numpy(g.r).to(dev)
    if g.pipe:
        u[2, :, 0, g.K] = (g.Re_i * (1 - r * r)).to(C128)
    else:
        u[1, :, 0, g.K] = (g.A * r + g.B / r).to(C128)
    if g.heated:
        u[3, :, 0, g.K] = (0.5 + torch.log(r / g.ri) / math.log(g.ri / g.ro)).to(C128)
    return u


def _inputs(case, seed, dev):
    """The input tensors of a case, from the seed alone."""
    g = _Geo(case)
    call = case["call"]
    if call == "remap":
        s = _Geo(case, case["from_N_r"], case["from_M_theta"], case["from_M_z"])
        return s, {"u": _base(s, dev) + _field(s, 4 * seed, dev, case["amp"])}
    d = {"u": _base(g, dev) + _field(g, 4 * seed, dev, case["amp"])}
    if call == "solve":  # nonlinear terms at the scale of the perturbation's
        scale = case["amp"] * max(abs(g.Re_i), 1.0)
        d["nn"] = _field(g, 4 * seed + 1, dev, scale, walls=False)
        d["nq"] = _field(g, 4 * seed + 2, dev, scale, walls=False)
    if call == "vjp":
        d["ubar"] = _field(g, 4 * seed + 3, dev, 1.0)
    return g, d


_ROWS, _THETA, _Z = (0.25, 0.5, 0.75), (0.0, 0.7, 2.1), (0.1, 1.3, 3.0)


def _context(case):
    import paper_1908_00587_amd as nsc
    if case["geometry"] == "pipe":
        ctx = nsc.Context.pipe(case["Re_i"], case["N_r"], case["M_theta"], case["M_z"], case["L_z"])
    else:
        ctx = nsc.Context(case["eta"], case["Re_i"], case["Re_o"], case["Ra"], case["Pr"],
                          case["N_r"], case["M_theta"], case["M_z"], case["L_z"])
    ctx.set_precision(case["precision"])
    return ctx


def prepare(case, seed):
    ctx = _context(case)
    g, s = _inputs(case, seed, "cuda")
    s.update(ctx=ctx, call=case["call"], dt=g.dt())
    ctx.set_timestep(dt=s["dt"], dynamic=case["dynamic"], cfl=0.5, dt_max=1e-3)
    call = case["call"]
    if call == "step":
        s.update(u0=s["u"].clone(), dt0=s["dt"], done=0)
    elif call == "solve":
        s.update(pressure=case.get("pressure", False), new_dt=case.get("new_dt", False))
    elif call == "vjp":
        from paper_1908_00587_amd import adjoint
        s["stages"], _ = adjoint.step_stages_fused(ctx, s["u"])
    elif call == "gradient":
        s.update(steps=case["steps"], ckpt=case["ckpt"])
    elif call == "monitor":
        s["rows"] = [int(x * (g.n - 1)) for x in _ROWS]
    return s


def run(s):
    ctx, call = s["ctx"], s["call"]
    if call == "step":  # the state is advanced in place, as a simulation does
        if s["done"] == 100:  # again from the same state, so that the flow stays the one described
            s["u"].copy_(s["u0"])
            s["dt"], s["done"] = s["dt0"], 0
        s["done"] += 1
        s["dt"] = ctx.step(s["u"], s["dt"])
        return {"u": s["u"], "dt": s["dt"]}
    if call == "nonlinear":
        n, cfl = ctx.nonlinear(s["u"], cfl=True)
        return {"n": n, "cfl": cfl}
    if call == "solve":
        if not s["new_dt"]:
            return _named(ctx.radial_solve(s["u"], s["nn"], s["nq"], pressure=s["pressure"]))
        out = {}
        for name, f in (("a", 1.0), ("b", 0.8)):
            ctx.set_timestep(dt=f * s["dt"])
            out[name] = _named(ctx.radial_solve(s["u"], s["nn"], s["nq"], pressure=s["pressure"]))
        return out
    if call == "vjp":
        from paper_1908_00587_amd import adjoint
        return adjoint.step_vjp_fused(ctx, s["u"], s["stages"], s["ubar"])
    if call == "gradient":
        from paper_1908_00587_amd import adjoint
        u = s["u"].detach().requires_grad_(True)
        e = adjoint.rollout_energy(ctx, u, s["steps"], s["dt"], ckpt_every=s["ckpt"])
        return {"energy": e.detach(), "grad": torch.autograd.grad(e, u)[0]}
    if call == "monitor":
        return {"energy": ctx.energy(s["u"]), "walls": ctx.diagnostics(s["u"]),
                "probes": ctx.probe(s["u"], s["rows"], _THETA, _Z)}
    return ctx.remap_state(s["u"])


def _named(r):
    return {"u": r[0], "p": r[1]} if isinstance(r, tuple) else {"u": r}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    g = _Geo(case)
    modes = g.Mt * g.Mz
    S = g.n * modes * 16.0  # one field
    n_in, n_out = (9, 4) if g.heated else (6, 3)
    lz, lt = math.log2(g.Nz), math.log2(g.Nt)
    nl = g.n * (n_in + n_out) * (g.Mt * 5.0 * g.Nz * lz + g.Nz * 2.5 * g.Nt * lt) + \
        30.0 * g.n * g.Nt * g.Nz
    ops = (g.K + 1.0) * g.n * 8
    fac = ops * (9 * (g.Mt + 1) + 9 * g.Mt * (2 if g.heated else 1) + 6 * g.Mt)  # LU rows, responses
    sol = modes * g.n * (4 + g.F) * 2 * 36.0
    call = case["call"]
    if call == "step":
        return {"bytes": 2 * g.F * S + fac, "flops": 2 * (nl + sol)}
    if call == "nonlinear":
        return {"bytes": 2 * g.F * S, "flops": nl}
    if call == "solve":
        b = 4 * g.F * S + (S if case.get("pressure") else 0)
        if case.get("new_dt"):
            return {"bytes": (3 * g.F + 2 * g.F) * S + 3 * fac, "flops": 2 * sol + 2 * fac / 8 * 12}
        return {"bytes": b + fac, "flops": sol}
    if call == "vjp":
        return {"bytes": 4 * g.F * S + fac, "flops": 2 * (2.2 * nl + sol)}
    if call == "gradient":
        k = case["steps"]
        return {"bytes": 2 * g.F * S + fac, "flops": k * 2 * (4.2 * nl + 3 * sol)}
    if call == "monitor":
        return {"bytes": g.F * S, "flops": 8 * modes * g.n}
    s = _Geo(case, case["from_N_r"], case["from_M_theta"], case["from_M_z"])
    kept = min(g.Mt, s.Mt) * min(g.Mz, s.Mz)
    return {"bytes": g.F * (S + 16.0 * s.n * kept), "flops": 4.0 * g.F * kept * g.n * s.n}


# ---------------------------------------------------------------------------
# plain FP64 values
# ---------------------------------------------------------------------------
def _weights(z, x):
    """Weights of the first and second derivative at z of the polynomial
    through the nodes x (B. Fornberg, Math. Comp. 51, 1988)."""
    x = [np.longdouble(v) for v in x]
    z = np.longdouble(z)
    n = len(x)
    w = np.zeros((n, 3), dtype=np.longdouble)
    w[0, 0] = 1
    c1 = np.longdouble(1)
    for i in range(1, n):
        c2 = np.longdouble(1)
        for j in range(i):
            c2 *= x[i] - x[j]
        for d in (2, 1, 0):
            low = d * w[i - 1, d - 1] if d else np.longdouble(0)
            w[i, d] = c1 * (low - (x[i - 1] - z) * w[i - 1, d]) / c2
        for j in range(i):
            for d in (2, 1, 0):
                low = d * w[j, d - 1] if d else np.longdouble(0)
                w[j, d] = ((x[i] - z) * w[j, d] - low) / (x[i] - x[j])
        c1 = c2
    return w[:, 1], w[:, 2]


class _Plain(_Geo):
    """The step in plain FP64: nine-point differences, FFTs on the 3/2-rule
    grid, dense solves per mode.  Index 0/1 of D1, D2: rows for functions
    even/odd in r (the pipe's mirror points; equal for the cylinders)."""

    def __init__(self, c):
        super().__init__(c)
        n, r = self.n, self.r
        D1, D2 = np.zeros((2, n, n)), np.zeros((2, n, n))
        for j in range(n):
            if self.pipe:  # nodes e = 0..2n-1 of [-1, 1], r_j at e = n + j
                s = min(n + j - 4, 2 * n - 9)
                cols = [(e - n, 1.0) if e >= n else (n - 1 - e, -1.0) for e in range(s, s + 9)]
            else:
                s = min(max(j - 4, 0), n - 9)
                cols = [(e, 1.0) for e in range(s, s + 9)]
            a, b = _weights(r[j], [sg * r[k] for k, sg in cols])
            for (k, sg), wa, wb in zip(cols, a, b):
                for odd in (0, 1):
                    f = sg if odd else 1.0
                    D1[odd, j, k] += f * float(wa)
                    D2[odd, j, k] += f * float(wb)
        self.D1, self.D2 = torch.from_numpy(D1), torch.from_numpy(D2)
        self.rt = torch.from_numpy(r)
        self.m = torch.arange(self.Mt, dtype=F64)[:, None]
        self.kap = (torch.arange(self.Mz, dtype=F64)[None, :] - self.K) * self.kz

    def d1(self, x, odd):
        """Radial derivative of [N_r][M_theta][M_z] coefficients of parity
        (-1)^(m + odd)."""
        if not self.pipe:
            return torch.tensordot(self.D1[0].to(C128), x, 1)
        y = torch.empty_like(x)
        for par in (0, 1):
            y[:, par::2] = torch.tensordot(self.D1[(par + odd) % 2].to(C128), x[:, par::2], 1)
        return y

    def herm(self, x):
        col = x[..., 0:1, :]
        return torch.cat([0.5 * (col + torch.flip(col, (-1,)).conj()), x[..., 1:, :]], dim=-2)

    def physical(self, f):  # one row [.., M_theta, M_z] -> [.., N_theta, N_z]
        K, Nz = self.K, self.Nz
        z = torch.zeros(f.shape[:-1] + (Nz - self.Mz,), dtype=C128)
        f = torch.fft.ifft(torch.cat([f[..., K:], z, f[..., :K]], -1), dim=-1, norm="forward")
        f = torch.cat([f, torch.zeros(f.shape[:-2] + (self.Nt // 2 + 1 - self.Mt, Nz), dtype=C128)], -2)
        return torch.fft.irfft(f, n=self.Nt, dim=-2, norm="forward")

    def spectral(self, f):
        h = torch.fft.fft(torch.fft.rfft(f, dim=-2)[..., :self.Mt, :], dim=-1) / (self.Nt * self.Nz)
        return torch.cat([h[..., self.Nz - self.K:], h[..., :self.K + 1]], -1)

    def nonlinear(self, u):
        """N(u) and the CFL bound; the mean flow is split off the products."""
        K = self.K
        mean = u[:, :, 0, K].real
        keep = torch.ones(self.Mt, self.Mz, dtype=F64)
        keep[0, K] = 0
        v = u * keep
        r3 = self.rt[:, None, None]
        imr, ik = 1j * self.m / r3, 1j * self.kap
        spec = [v[0], v[1], v[2], imr * v[2] - ik * v[1], ik * v[0] - self.d1(v[2], 0),
                self.d1(v[1], 1) + v[1] / r3 - imr * v[0]]
        if self.heated:
            spec += [self.d1(v[3], 0), imr * v[3], ik * v[3]]
        spec = torch.stack(spec)
        odd = 1 if self.pipe else 0
        Ur, V, W = mean[0], mean[1], mean[2]
        Ot, Oz = -(self.D1[0] @ W), self.D1[odd] @ V + V / self.rt
        G = self.D1[0] @ mean[3] if self.heated else None
        dr = np.diff(self.r)
        lo = np.concatenate([[2 * self.r[0] if self.pipe else dr[0]], dr])
        dr = np.minimum(lo, np.concatenate([dr, dr[-1:]]))
        rows, cfl = [], math.inf
        for j in range(self.n):
            a = self.physical(spec[:, j])
            ur, ut, uz, wr, wt, wz = a[:6]
            o = [ut * wz - uz * wt + V[j] * wz - W[j] * wt + ut * Oz[j] - uz * Ot[j],
                 uz * wr - ur * wz + W[j] * wr - Ur[j] * wz - ur * Oz[j],
                 ur * wt - ut * wr + Ur[j] * wt - V[j] * wr + ur * Ot[j]]
            if self.heated:
                gr, gt, gz = a[6:9]
                o.append(-(ur * gr + ut * gt + uz * gz + Ur[j] * gr + V[j] * gt + W[j] * gz + ur * G[j]))
            rows.append(self.spectral(torch.stack(o)))
            with torch.no_grad():
                for f, mn, h in ((ur, Ur, dr[j]), (ut, V, self.r[j] * TWO_PI / self.Nt),
                                 (uz, W, self.Lz / self.Nz)):
                    top = float((f + mn[j]).abs().max())
                    cfl = min(cfl, h / top) if top > 0 else cfl
        N = torch.stack(rows, 1)
        add = [V * Oz - W * Ot, -Ur * Oz, Ur * Ot] + ([-Ur * G] if self.heated else [])
        hot = torch.zeros(self.Mt, self.Mz, dtype=C128)
        hot[0, K] = 1
        N = N + torch.stack(add)[:, :, None, None] * hot
        if self.heated:
            gt = torch.zeros_like(N)
            gt[2] = self.Ra / self.Pr
            N = N + gt * u[3]
        return self.herm(N), cfl

    def _lap(self, q, kap):
        """L_q of each mode, [B][n][n]."""
        D = (self.D2 + self.D1 / self.rt[:, None])[(q % 2).long()]
        return D - torch.diag_embed(q[:, None] ** 2 / self.rt ** 2 + kap[:, None] ** 2)

    def solve(self, u, nn, nq, dt, c=0.5, want_p=False):
        n, B, K = self.n, self.Mt * self.Mz, self.K
        flat = lambda x: x.reshape(n, B).T  # noqa: E731
        wall = [n - 1] if self.pipe else [0, n - 1]
        inner = torch.ones(n, dtype=F64)
        inner[wall] = 0
        eye = torch.eye(n, dtype=F64)
        out = {k: [] for k in ("r", "t", "z", "p", "T")}
        step = max(1, min(B, 2 ** 25 // (n * n)))
        X = [flat(u[f]) for f in range(self.F)]
        Nc = [c * flat(nq[f]) + (1 - c) * flat(nn[f]) for f in range(self.F)]
        mall = self.m.expand(self.Mt, self.Mz).reshape(-1)
        kall = self.kap.expand(self.Mt, self.Mz).reshape(-1)

        def app(A, x):
            return torch.complex((A @ x.real[..., None])[..., 0], (A @ x.imag[..., None])[..., 0])

        def inv(A, xs):
            s = torch.linalg.solve(A, torch.stack([y for x in xs for y in (x.real, x.imag)], -1))
            return [torch.complex(s[..., 2 * i], s[..., 2 * i + 1]) for i in range(len(xs))]

        for b0 in range(0, B, step):
            sl = slice(b0, min(B, b0 + step))
            m, kap = mall[sl], kall[sl]
            nb = m.numel()
            zero = (torch.arange(sl.start, sl.stop) == K)[:, None]
            ri = 1 / self.rt[None, :]
            Dm, Dq = self.D1[(m % 2).long()], self.D1[((m + 1) % 2).long()]
            Lp, Lm, Lz = self._lap(m + 1, kap), self._lap((m - 1).abs(), kap), self._lap(m, kap)
            xr, xt, xz = (x[sl] for x in X[:3])
            ar, at, az = (x[sl] for x in Nc[:3])
            xp, xm = xr + 1j * xt, xr - 1j * xt
            fp = xp / dt + (1 - c) * app(Lp, xp) + ar + 1j * at
            fm = xm / dt + (1 - c) * app(Lm, xm) + ar - 1j * at
            fz = xz / dt + (1 - c) * app(Lz, xz) + az

            def div(p, q, z):
                return 0.5 * (app(Dq, p) + (1 + m)[:, None] * ri * p + app(Dq, q) +
                              (1 - m)[:, None] * ri * q) + 1j * kap[:, None] * z

            def boundary(A, rows):
                A = A * inner[:, None]
                for w in wall:
                    A = A + torch.zeros_like(A).index_add(
                        -2, torch.tensor([w]), rows[..., w:w + 1, :].expand(nb, 1, n))
                return A

            g = div(fp, fm, fz) * inner * (~zero)
            # pressure and its responses to unit wall data; mode (0,0): the
            # mean head, (D2 + D1/r) p = (D1 + 1/r) F_r
            P = boundary(Lz, Dm)
            fr = ar
            head = app(Dq, fr) + ri * fr
            if self.pipe:
                P00 = boundary(Lz, eye[None])
                rhs00 = head * inner
            else:
                rows = torch.cat([eye[None, :1], Dm[:1, 1:]], 1)
                P00 = boundary(Lz, rows.expand(nb, n, n))
                rhs00 = head * inner + fr * eye[-1]
            P = torch.where(zero[:, :, None], P00, P)
            es = [eye[w].to(C128).expand(nb, n) for w in wall]
            ps = inv(P, [torch.where(zero, rhs00, g)] + es)
            Hp, Hm, Hz = (boundary(eye / dt - c * L, eye[None]) for L in (Lp, Lm, Lz))
            rp, rm, rz = [], [], []
            for i, p in enumerate(ps):
                dp, mp = app(Dm, p), m[:, None] * ri * p
                s = 1.0 if i == 0 else 0.0
                rp.append((s * fp - (dp - mp) * (~zero)) * inner)
                rm.append((s * fm - (dp + mp) * (~zero)) * inner)
                rz.append((s * fz - 1j * kap[:, None] * p * (~zero)) * inner)
            # mode (0,0): u_theta and u_z directly, wall speeds
            ut0 = 0.5 * (fp - fm) * inner
            if not self.pipe:
                ut0 = ut0 + 1j * (self.Re_i * eye[0] + self.Re_o * eye[-1])
            else:
                rz[0] = rz[0] + zero * inner * (4 * self.Re_i)
            rp[0] = torch.where(zero, ut0, rp[0])
            rm[0] = torch.where(zero, -ut0, rm[0])
            sp, sm, sz = inv(Hp, rp), inv(Hm, rm), inv(Hz, rz)
            beta = [div(a, b, z)[:, wall] for a, b, z in zip(sp, sm, sz)]
            A = torch.stack([b.real for b in beta[1:]], -1)
            A = torch.where(zero[:, :, None], torch.eye(len(wall), dtype=F64), A)
            lam = -torch.linalg.solve(A.to(C128), beta[0][..., None])[..., 0] * (~zero)
            for i in range(len(wall)):
                l = lam[:, i:i + 1]
                sp[0], sm[0], sz[0] = sp[0] + l * sp[i + 1], sm[0] + l * sm[i + 1], sz[0] + l * sz[i + 1]
                ps[0] = ps[0] + l * ps[i + 1]
            out["r"].append(0.5 * (sp[0] + sm[0]))
            out["t"].append(-0.5j * (sp[0] - sm[0]))
            out["z"].append(sz[0])
            out["p"].append(ps[0])
            if self.heated:
                xT, LT = X[3][sl], Lz / self.Pr
                fT = (xT / dt + (1 - c) * app(LT, xT) + Nc[3][sl]) * inner
                fT = fT + zero * (0.5 * eye[0] - 0.5 * eye[-1])
                out["T"].append(inv(boundary(eye / dt - c * LT, eye[None]), [fT])[0])
        back = lambda k: torch.cat(out[k]).T.reshape(n, self.Mt, self.Mz)  # noqa: E731
        new = self.herm(torch.stack([back(k) for k in ("r", "t", "z", "T")[:self.F]]))
        return (new, self.herm(back("p"))) if want_p else new

    def step(self, u, dt):
        nn, cfl = self.nonlinear(u)
        x = self.solve(u, nn, nn, dt)
        return self.solve(u, nn, self.nonlinear(x)[0], dt), cfl

    def energy(self, u):
        n = self.n
        j = np.arange(n)
        V = np.cos(np.pi * np.outer(j, n - 1 - j) / (n - 1))
        mom = np.array([2 / (1 - k * k) if k % 2 == 0 else 0.0 for k in j])
        w = torch.from_numpy(0.5 * np.linalg.solve(V, mom)) * self.rt
        d = (u - _base(self, "cpu"))[:3]
        cm = torch.full((self.Mt, 1), 2.0, dtype=F64)
        cm[0] = 1
        return math.pi * self.Lz * (w[:, None, None] * cm * (d.real ** 2 + d.imag ** 2)).sum()


def exact(case, seed):
    call = case["call"]
    g = _Geo(case)
    modes, pts = g.Mt * g.Mz, g.n * g.Nt * g.Nz
    dense = modes * float(g.n) ** 3 * (5 if g.heated else 4)
    grad = {"vjp": 5, "gradient": 6 * case.get("steps", 1)}.get(call, 1)
    halves = {"step": 2, "vjp": 2, "gradient": 2, "solve": 1 + case.get("new_dt", False)}.get(call, 0)
    if halves * grad * dense > 5e10 or (call not in ("solve", "monitor", "remap") and grad * pts > 6e7):
        return None
    geo, d = _inputs(case, seed, "cuda")
    d = {k: v.cpu() for k, v in d.items()}
    u, dt = d["u"], g.dt()
    if call == "remap":
        return _remap(geo, g, u)
    p = _Plain(case)
    if call == "step":
        return {"u": p.step(u, dt)[0], "dt": None}
    if call == "nonlinear":
        n, cfl = p.nonlinear(u)
        return {"n": n, "cfl": torch.tensor([cfl], dtype=F64)}
    if call == "solve":
        def one(h):
            return _named(p.solve(u, d["nn"], d["nq"], h, want_p=case.get("pressure", False)))
        return {"a": one(dt), "b": one(0.8 * dt)} if case.get("new_dt") else one(dt)
    if call == "vjp":
        u.requires_grad_(True)
        return torch.autograd.grad(p.step(u, dt)[0], u, d["ubar"])[0]
    if call == "gradient":
        x = u.requires_grad_(True)
        for _ in range(case["steps"]):
            x = p.step(x, dt)[0]
        e = p.energy(x)
        return {"energy": e.detach().reshape(1), "grad": torch.autograd.grad(e, u)[0]}
    m = u[:, :, 0, g.K].real
    dv = p.D1[0] @ m[1]
    torque = -TWO_PI * g.Lz * (p.rt ** 2 * dv - p.rt * m[1])
    nus = p.rt * math.log(g.eta) * (p.D1[0] @ m[3]) if g.heated else torch.zeros(g.n, dtype=F64)
    probes = []
    for x, th, z in zip(_ROWS, _THETA, _Z):
        ph = torch.exp(1j * (p.m * th + p.kap * z)) * torch.where(p.m == 0, 1.0, 2.0)
        probes.append((u[:, int(x * (g.n - 1))] * ph).real.sum((1, 2)))
    return {"energy": p.energy(u).reshape(1), "probes": torch.stack(probes),
            "walls": torch.stack([nus[0], nus[-1], torque[0], torque[-1]])}


def _remap(s, g, u):
    """Modes kept, the radial profile through all old points."""
    w = (-1.0) ** np.arange(s.n)
    w[[0, -1]] *= 0.5
    W = np.zeros((g.n, s.n))
    for i, r in enumerate(g.r):
        near = np.abs(r - s.r) < 1e-14 * r
        if near.any():
            W[i, near.argmax()] = 1
        else:
            W[i] = w / (r - s.r) / (w / (r - s.r)).sum()
    out = torch.zeros(g.shape(), dtype=C128)
    Mt, K = min(g.Mt, s.Mt), min(g.K, s.K)
    new = torch.einsum("ij,fjmk->fimk", torch.from_numpy(W).to(C128),
                       u[:, :, :Mt, s.K - K:s.K + K + 1].contiguous())
    out[:, :, :Mt, g.K - K:g.K + K + 1] = new
    return out
