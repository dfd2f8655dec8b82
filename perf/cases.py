"""What a user of the library has it do, as cases that can be timed.

Every case goes through paper_1706_07413_amd.adscl, from data in hand (grid
sizes, amplitudes, mode coefficients) to the arrays a study works with: states
and their metric, spectra, diagnostics, gradients.  Four kinds:

  evolve    initial data, a window of RK steps (with snapshots where asked) and
            the state, the status and, of the snapshots, the mode energies;
  monitor   a few further steps of a run, its status and its diagnostics;
  analyse   mode energies and diagnostics of the current states;
  adjoint   one gradient of the drift objective, or some descent iterations.

`exact` evaluates the same discrete equations with torch tensors in 64 bits
(the gradient by torch's own autograd), without the library.
"""
import math

import numpy as np
import torch

from paper_1706_07413_amd import adscl, inputs

BASE = dict(kind="evolve", n_inst=1, grid="one", n=1025, n_top=0, grid_seed=0, data="gaussian", eps_lo=1.0, eps_hi=10.0,
            sig_lo=1.0 / 16.0, sig_hi=1.0 / 4.0, n_modes=0, coefs=0, steps=256, snap_every=0, gauge="boundary", rk=4, a_reint=0, frozen=False,
            T=0.0, ckpt=512, iters=0, a_collapse=0.01)

# Algorithmic flops of one grid point in one right-hand side, counted from the
# scheme (bench.py), and of its transpose (every add and multiply again, and the
# products' second factors).
FLOPS_STAGE, FLOPS_REVERSE = 67.0, 150.0


def _case(name, **kw):
    assert set(kw) <= set(BASE), kw
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # a run followed live: some steps, then status and residuals, again and again
        _case("monitor_n1025", kind="monitor", n=1025, steps=16, eps_lo=2.0, eps_hi=8.0),
        # the small single run with its snapshots, origin time, t = pi: out to the boundary and back
        _case("gaussian_n513_snaps", n=513, steps=4096, snap_every=256, gauge="origin", eps_lo=9.0, eps_hi=10.0,
              sig_hi=1.0 / 15.0),
        # the batched Gaussian study: 1024 instances on three grids
        _case("gaussian_batch_1024", n_inst=1024, grid="mix", n=1025, n_top=4097, eps_lo=1.0, eps_hi=40.0, steps=512,
              a_collapse=0.02),
        # a resolution scan: grids of any odd size, few of which fill whole wavefronts
        _case("ragged_batch_192", n_inst=192, grid="ragged", n=17, n_top=4095, grid_seed=1, eps_lo=1.0, eps_hi=10.0,
              steps=512),
        # the collapse-time sweep of the quasi-periodic families, the paper's third-order integrator
        _case("qp_64_n4097_rk3", n_inst=64, n=4097, data="qp", eps_lo=0.006, eps_hi=0.04, n_modes=40, coefs=40, rk=3,
              steps=1024),
        # the same sweep at twice the resolution (several workgroups per instance, the whole device busy)
        _case("qp_64_n8193_rk3", n_inst=64, n=8193, data="qp", eps_lo=0.006, eps_hi=0.04, n_modes=40, coefs=40, rk=3,
              steps=512),
        # the long two-mode run with its spectra, one large instance
        _case("twomode_n16385_spec", n=16385, data="modes", eps_lo=0.04, eps_hi=0.06, n_modes=64, coefs=2, steps=2048,
              snap_every=512),
        # the paper's speed-table grid, dynamic metric
        _case("table_n32769", n=32769, eps_lo=1.0, eps_hi=3.0, steps=512),
        # the paper's speed-table grid, metric frozen
        _case("table_n65537_frozen", n=65537, eps_lo=1.0, eps_hi=3.0, steps=512, frozen=True),
        # spectra and residuals of a batch's current states
        _case("analyse_batch_1024", kind="analyse", n_inst=1024, grid="mix", n=1025, n_top=4097, n_modes=32, eps_lo=1.0,
              eps_hi=6.0),
        # one gradient of the drift objective
        _case("adjoint_n4097", kind="adjoint", n=4097, data="modes", eps_lo=0.1, eps_hi=0.12, n_modes=32, coefs=32,
              T=0.1),
        # batched gradient descent: 256 instances on two grids, two iterations
        _case("descend_batch_256", kind="adjoint", n_inst=256, grid="mix", n=2049, n_top=4097, data="modes", eps_lo=0.02,
              eps_hi=0.2, n_modes=32, coefs=32, T=0.1, iters=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, lo, hi):
    return min(hi, max(lo, _log_int(rng, lo, hi) | 1))


def draw(rng):
    """One more case of the same ranges: full grids (a power of two plus one)
    and odd ones in between, every scheme option, from one instance to a
    thousand."""
    full = [257, 513, 1025, 2049, 4097]
    kind = rng.choice(["monitor", "single", "batch", "ragged", "qp", "large", "large", "frozen", "analyse", "gradient",
                       "descent"])
    n = rng.choice(full) if rng.random() < 0.6 else _odd(rng, 129, 4095)
    gauge = rng.choice(["boundary", "boundary", "origin"])
    c = dict(BASE, grid_seed=rng.randrange(1 << 16))
    if kind == "monitor":
        c.update(kind="monitor", n=n, n_inst=_log_int(rng, 1, 64), steps=_log_int(rng, 1, 64), eps_lo=1.0, eps_hi=8.0)
    elif kind == "single":
        k = _log_int(rng, 64, 512)
        c.update(n=n, steps=_log_int(rng, 512, 4096), snap_every=rng.choice([0, k]), gauge=gauge, eps_lo=1.0, eps_hi=8.0)
    elif kind == "batch":
        c.update(n_inst=_log_int(rng, 16, 1000), grid="mix", n=rng.choice([513, 1025]), n_top=rng.choice([2049, 4097]),
                 steps=_log_int(rng, 128, 500), eps_hi=20.0, a_collapse=0.02)
    elif kind == "ragged":
        c.update(n_inst=_log_int(rng, 2, 190), grid="ragged", n=17, n_top=_odd(rng, 513, 4095),
                 steps=_log_int(rng, 128, 500), gauge=gauge, frozen=rng.random() < 0.2, eps_hi=6.0)
    elif kind == "qp":
        rk = rng.choice([2, 3, 3, 4])
        c.update(n_inst=_log_int(rng, 4, 64), n=rng.choice([1025, 2049, 4097]), data="qp", eps_lo=0.006, eps_hi=0.04,
                 n_modes=40, coefs=40, rk=rk, a_reint=rng.choice([0, 0, 4, 16]), steps=_log_int(rng, 128, 1000))
    elif kind == "large":
        n = rng.choice([8193, 16385, 32769]) if rng.random() < 0.6 else _odd(rng, 6001, 40001)
        while (n - 1) % 2048 and (n - 1) % 2048 < 16:
            n += 16
        c.update(n=n, n_inst=rng.choice([1, 1, 2, 5]), steps=_log_int(rng, 128, 500), rk=rng.choice([3, 4, 4]),
                 a_reint=rng.choice([0, 0, 0, 16]), gauge=gauge, eps_lo=1.0, eps_hi=3.0)
    elif kind == "frozen":
        c.update(n=rng.choice([4097, 16385, 32769, 65537]), steps=_log_int(rng, 128, 500), frozen=True, eps_hi=3.0)
    elif kind == "analyse":
        c.update(kind="analyse", n_inst=_log_int(rng, 1, 1000), n=n, n_modes=rng.choice([8, 16, 32, 33]), eps_hi=6.0)
    elif kind == "gradient":
        c.update(kind="adjoint", n=rng.choice([513, 1025, 2049, 4097, n]), n_inst=_log_int(rng, 1, 16), data="modes",
                 eps_lo=0.1, eps_hi=0.2, n_modes=32, coefs=_log_int(rng, 2, 32), T=rng.uniform(0.05, 0.1),
                 ckpt=_log_int(rng, 64, 512))
    else:
        assert kind == "descent"
        c.update(kind="adjoint", n_inst=_log_int(rng, 16, 250), grid="mix", n=rng.choice([513, 1025, 2049]), n_top=4097,
                 data="modes", eps_lo=0.1, eps_hi=0.2, n_modes=16, coefs=16, T=rng.uniform(0.05, 0.09), iters=2)
    if c["gauge"] == "origin":
        # in origin time the speed at the boundary grows with the mass, and with it the stable step shrinks
        c.update(eps_hi=min(c["eps_hi"], 3.0), sig_hi=1.0 / 8.0)
    return c


# ---- inputs -----------------------------------------------------------------

def _grids(case):
    n = case["n_inst"]
    r = np.random.default_rng(inputs.SEED_BASE + case["grid_seed"])
    if case["grid"] == "one":
        return np.full(n, case["n"], np.int32)
    if case["grid"] == "mix":
        sizes, k = [], case["n"]
        while k <= case["n_top"]:
            sizes.append(k)
            k = 2 * k - 1
        return r.choice(np.array(sizes, np.int32), size=n).astype(np.int32)
    return (2 * r.integers(case["n"] // 2, case["n_top"] // 2 + 1, size=n) + 1).astype(np.int32)


def _data(case, seed):
    """eps [n], sigma [n] or None, coefficients [n, coefs] or None."""
    n = case["n_inst"]
    r = np.random.default_rng([inputs.SEED_BASE, seed, n])
    eps = np.exp(r.uniform(math.log(case["eps_lo"]), math.log(case["eps_hi"]), size=n))
    if case["data"] == "gaussian":
        return eps, r.uniform(case["sig_lo"], case["sig_hi"], size=n), None
    if case["data"] == "qp":
        fam = [inputs.qp_family(kd, mu, case["coefs"]) for kd, mu in inputs.QP_FAMILIES]
        return eps, None, np.ascontiguousarray(np.stack([fam[b % 4] for b in range(n)]))
    return eps, None, np.ascontiguousarray(inputs.mode_coefficients(r, n, case["coefs"]))


def _flags(case):
    return adscl.FROZEN_METRIC if case["frozen"] else 0


def prepare(case, seed):
    N = _grids(case)
    eps, sigma, c = _data(case, seed)
    b = adscl.Batch(N, a_collapse=case["a_collapse"], n_modes=case["n_modes"], flags=_flags(case), rk_order=case["rk"],
                    a_reint=case["a_reint"],
                    gauge=adscl.GAUGE_ORIGIN if case["gauge"] == "origin" else adscl.GAUGE_BOUNDARY)
    s = dict(case=case, batch=b, eps=eps, sigma=sigma, c=c)
    if case["kind"] == "adjoint":
        s["eps"] = torch.from_numpy(eps).cuda()
        s["c"] = torch.from_numpy(c).cuda()
        return s
    if case["kind"] in ("monitor", "analyse"):
        # the run is under way: its state is at a later step
        _init(s)
        b.step(64, 1e9)
        st = b.get_state()
        s["Phi"], s["Pi"] = st["Phi"], st["Pi"]
        b.init(s["Phi"], s["Pi"])
    if case["snap_every"]:
        slots = case["steps"] // case["snap_every"] + 1
        s["snaps"] = torch.zeros((slots, 5, b.total), dtype=torch.float64, device="cuda")
    s["out"] = {k: torch.empty(b.total, dtype=torch.float64, device="cuda") for k in ("Phi", "Pi", "A", "delta", "m")}
    return s


def _init(s):
    if s["sigma"] is not None:
        s["batch"].init_gaussian(s["eps"], s["sigma"])
    else:
        s["batch"].init_modes(s["eps"], s["c"])


def run(s):
    case, b = s["case"], s["batch"]
    if case["kind"] == "adjoint":
        if case["iters"]:
            c, hist, active = b.descend(s["eps"], s["c"], 16, case["T"], case["iters"], ckpt_every=case["ckpt"])
            return dict(c=c, L_hist=hist, active=active)
        L, g, valid = b.adjoint(s["eps"], s["c"], 16, case["T"], case["ckpt"])
        return dict(L=L, dLdc=g, valid=valid)
    if case["kind"] == "analyse":
        E, P, F = b.spectrum(case["n_modes"])
        return dict(E=E, Pihat=P, Phihat=F, residuals=b.constraints())
    if case["kind"] == "monitor":
        b.init(s["Phi"], s["Pi"])
        b.step(case["steps"], 1e9)
        return dict(status=b.status(), residuals=b.constraints())
    _init(s)
    snaps = s.get("snaps")
    b.step(case["steps"], 1e9, case["snap_every"], snaps)
    out = dict(status=b.status(), state=b.get_state(s["out"]))
    if snaps is not None:
        out["snaps"] = snaps
        if case["n_modes"]:
            out["spectra"] = b.spectrum_snaps(case["n_modes"], snaps)
    return out


def _n_steps(N, T):
    return np.ceil(T / (0.25 * (math.pi / 2) / (N - 1)) - 1e-9).astype(np.int64)


def work(case):
    N = _grids(case).astype(np.float64)
    total, n = float(N.sum()), case["n_inst"]
    stages = case["rk"]
    J = case["n_modes"]
    if case["kind"] == "adjoint":
        steps = float((N * _n_steps(N, case["T"])).sum()) * 4 * max(1, case["iters"])
        return dict(bytes=8.0 * (2 * n * case["coefs"] + 3 * n), flops=steps * (FLOPS_STAGE + FLOPS_REVERSE))
    # states read once (Phi, Pi, A, delta, m) and, per projected state, two products of length N with J modes
    if case["kind"] == "analyse":
        return dict(bytes=8.0 * (5 * total + 2 * J * len(set(N)) * N.max() + 3 * n * J), flops=total * (4.0 * J + 80.0))
    flops = total * stages * case["steps"] * FLOPS_STAGE
    if case["kind"] == "monitor":
        return dict(bytes=8.0 * (2 * total + 10 * n), flops=flops)
    slots = case["steps"] // case["snap_every"] + 1 if case["snap_every"] else 0
    return dict(bytes=8.0 * total * 5 * (1 + slots), flops=flops + slots * total * 4.0 * J)


# ---- the same equations with torch tensors in 64 bits -----------------------

def _modes(N, J):
    """e_j(x_i), h tan^2 x e_j and h tan^2 x e_j'/omega_j, [J, N] each."""
    ld = np.longdouble
    pi = ld("3.14159265358979323846264338327950288")
    h = pi / 2 / (N - 1)
    x = h * np.arange(N, dtype=ld)
    s, c = np.sin(x), np.cos(x)
    s[-1], c[-1] = 1, 0
    z = c * c - s * s

    def jacobi(a, b):
        a, b = ld(a), ld(b)
        out = [np.ones_like(z), ld(0.5) * ((a + b + 2) * z + (a - b))]
        for m in range(2, J + 1):
            k = 2 * m + a + b
            out.append(((k - 1) * (k * (k - 2) * z + a * a - b * b) * out[-1] - 2 * (m + a - 1) * (m + b - 1) * k * out[-2])
                       / (2 * m * (m + a + b) * (k - 2)))
        return out

    P, Q = jacobi(0.5, 1.5), jacobi(1.5, 2.5)
    t2 = np.zeros_like(x)
    t2[1:-1] = (s[1:-1] / c[1:-1]) ** 2
    e, wpi, wphi = (np.zeros((J, N)) for _ in range(3))
    for j in range(J):
        # lgamma in 64 bits loses digits; the same factor as a product: d_j^2 = 4 j! (j+2)! / Gamma(j+3/2)^2
        d2 = ld(8) * 4 / pi
        for i in range(1, j + 1):
            d2 *= ld(i) * (i + 2) / ((ld(i) + ld(0.5)) ** 2)
        d = np.sqrt(d2)
        ej = d * c ** 3 * P[j]
        dP = ld(0.5) * (j + 3) * Q[j - 1] if j else 0 * z
        dej = d * (-3 * c * c * s * P[j] - 4 * s * c ** 4 * dP)
        e[j], wpi[j], wphi[j] = ej, h * t2 * ej, h * t2 * dej / (3 + 2 * j)
    return e, wpi, wphi


class _Exact:
    """The semi-discrete system of a padded batch [B, N_max]: points past an
    instance's end hold zeros, ghosts are gathered from their mirror points."""

    def __init__(self, N, case, dev):
        self.N, self.dev = N, dev
        B, M = len(N), int(N.max())
        i = np.arange(M)
        n1 = (N - 1)[:, None].astype(np.longdouble)
        pi = np.longdouble("3.14159265358979323846264338327950288")
        x = pi / 2 * i[None, :] / n1
        inner = (i[None, :] >= 1) & (i[None, :] <= N[:, None] - 2)
        x = np.where(inner, x, 1)
        s, c = np.sin(x), np.cos(x)

        def t(a):
            return torch.from_numpy(np.where(inner, a, 0).astype(np.float64)).to(dev)

        self.sc, self.t2, self.ct2, self.c3s = t(s * c), t((s / c) ** 2), t((c / s) ** 2), t(c ** 3 / s)
        self.s2 = t(s * s)
        self.inner = torch.from_numpy(inner).to(dev)
        self.live = torch.from_numpy(i[None, :] <= N[:, None] - 2).to(dev)
        self.m0, self.m1 = self.inner.double(), self.live.double()
        self.at0 = torch.from_numpy(i[None, :] == 0).to(dev)
        self.atN = torch.from_numpy(i[None, :] == N[:, None] - 1).double().to(dev)
        h = (math.pi / 2) / (N - 1)
        col = lambda a: torch.from_numpy(np.asarray(a, np.float64)[:, None]).to(dev)  # noqa: E731
        self.h, self.dt = col(h), col(0.25 * h)
        self.k = col(0.5 / (64.0 * h))
        self.n1 = torch.from_numpy((N - 1).astype(np.int64)[:, None]).to(dev)
        self.idx, self.sgn = {}, {}
        for g in (1, 2, 3):
            j = np.arange(-g, M + g)[None, :].repeat(B, 0)
            left, right = j < 0, j > (N - 1)[:, None]
            j = np.where(right, 2 * (N - 1)[:, None] - j, np.abs(j))
            far = j < np.maximum(0, (N - 1)[:, None] - g) * right
            j = np.where(far | (j < 0), 0, j)
            self.idx[g] = torch.from_numpy(j).to(dev)
            for name, l, r in (("eo", 1.0, -1.0), ("oe", -1.0, 1.0), ("oo", -1.0, -1.0), ("ee", 1.0, 1.0)):
                w = np.where(left, l, np.where(right, r, 1.0)) * np.where(far, 0.0, 1.0)
                self.sgn[g, name] = torch.from_numpy(w).to(dev)
        self.frozen, self.boundary, self.thr = case["frozen"], case["gauge"] == "boundary", case["a_collapse"]

    def ext(self, u, g, parity):
        return u.gather(1, self.idx[g]) * self.sgn[g, parity]

    def cell(self, u, parity):
        v = self.ext(u, 1, parity)
        return self.h / 24 * (24 * u.cumsum(1) - 12 * u + v[:, :-2] - v[:, 2:])

    def solve(self, q):
        """delta before the shift, the shift, e^-delta, S."""
        p = self.sc * q
        d = -self.cell(p, "oo") - self.h / 12 * p[:, 1:2]
        shift = d.gather(1, self.n1) if self.boundary else torch.zeros_like(d[:, :1])
        E = torch.exp(shift - d)
        return d, shift, E, self.cell(self.t2 * q * E, "ee")

    def rhs(self, U, V, A=None):
        """Phi_t, Pi_t, w = A e^-delta, e^-delta; A given: evolved, not solved."""
        q = U * U + V * V
        if self.frozen:
            E = w = torch.ones_like(q)
        else:
            d, shift, E, S = self.solve(q)
            w = E - self.c3s * S if A is None else A * E
        f1, f2 = w * V, w * U
        g = self.t2 * f2
        ge = (15 * g.gather(1, self.n1 - 1) - 6 * g.gather(1, self.n1 - 2) + g.gather(1, self.n1 - 3)) / 10
        e1, e2 = self.ext(f1 * self.m1, 2, "eo"), self.ext(g + self.atN * ge, 2, "oe")
        i12 = 1 / (12 * self.h)
        d1 = (e1[:, :-4] - 8 * e1[:, 1:-3] + 8 * e1[:, 3:-1] - e1[:, 4:]) * i12
        d2 = (e2[:, :-4] - 8 * e2[:, 1:-3] + 8 * e2[:, 3:-1] - e2[:, 4:]) * i12
        o = 3 * ((16 * f2[:, 1:2] - 2 * f2[:, 2:3]) * i12)
        r0 = (d1 + self.k * torch.diff(self.ext(U, 3, "oe"), n=6)) * self.m0
        r1 = (torch.where(self.at0, o, self.ct2 * d2) + self.k * torch.diff(self.ext(V, 3, "eo"), n=6)) * self.m1
        return r0, r1, w, E

    def A_of(self, q):
        if self.frozen:
            return torch.ones_like(q)
        d, shift, E, S = self.solve(q)
        return 1 - self.c3s * (S / E)

    def step4(self, U, V, dt):
        a, b, w, E = self.rhs(U, V)
        sa, sb = a, b
        for f, k in ((0.5, 2), (0.5, 2), (1.0, 1)):
            a, b, _, _ = self.rhs(U + f * dt * a, V + f * dt * b)
            sa, sb = sa + k * a, sb + k * b
        return U + dt / 6 * sa, V + dt / 6 * sb, w, E

    def evolve(self, U, V, steps, rk, K, snap=None, snap_every=0):
        """Runs `steps` steps; instances stop where min A falls below the
        threshold.  Returns U, V and the evolved A (None where A is solved)."""
        dt, A = self.dt, None
        alive = torch.ones_like(dt, dtype=torch.bool)
        for n in range(steps):
            if snap and n % snap_every == 0:
                snap(n, U, V)
            if K and n % K == 0:
                A = self.A_of(U * U + V * V)
            U0, V0, A0 = U, V, A
            if rk == 4 and not K:
                U, V, w, E = self.step4(U, V, dt)
            else:
                def f(u, v, a):
                    r0, r1, w_, E_ = self.rhs(u, v, a)
                    return r0, r1, None if a is None else -2 * self.sc * a * w_ * u * v, w_, E_

                def add(x, c, y):
                    return None if x is None else x + c * y

                x = (U, V, A)
                *k1, w, E = f(*x)
                if rk == 4:
                    acc = k1
                    k = k1
                    for c, m in ((0.5, 2), (0.5, 2), (1.0, 1)):
                        *k, _, _ = f(*(add(x[i], c * dt, k[i]) for i in range(3)))
                        acc = [add(acc[i], m, k[i]) for i in range(3)]
                    y = [add(x[i], dt / 6, acc[i]) for i in range(3)]
                else:
                    y = [add(x[i], dt, k1[i]) for i in range(3)]
                    *k2, _, _ = f(*y)
                    z = [add(y[i], dt, k2[i]) for i in range(3)]
                    if rk == 2:
                        y = [None if z[i] is None else 0.5 * x[i] + 0.5 * z[i] for i in range(3)]
                    else:
                        y = [None if z[i] is None else 0.75 * x[i] + 0.25 * z[i] for i in range(3)]
                        *k3, _, _ = f(*y)
                        y = [None if y[i] is None else x[i] / 3 + 2.0 / 3.0 * (y[i] + dt * k3[i]) for i in range(3)]
                U, V, A = y
            alive = alive & ~((w < self.thr * E) & self.live).any(1, keepdim=True)
            U, V = torch.where(alive, U, U0), torch.where(alive, V, V0)
            if A is not None:
                A = torch.where(alive, A, A0)
        if snap and steps % snap_every == 0:
            snap(steps, U, V)
        self.alive = alive
        return U, V, A

    def metric(self, U, V, A=None):
        q = U * U + V * V
        if self.frozen:
            return torch.ones_like(q), torch.zeros_like(q), torch.zeros_like(q)
        d, shift, E, S = self.solve(q)
        m = S / E
        return (1 - self.c3s * m) if A is None else A, d - shift, m

    def pack(self, a):
        return torch.cat([a[b, :n] for b, n in enumerate(self.N.tolist())])

    def energies(self, U, V, A, tabs):
        """E, Pihat, Phihat [B, J]."""
        rA = torch.sqrt(A)
        P, F = [], []
        for b, n in enumerate(self.N.tolist()):
            _, wpi, wphi = tabs[n]
            P.append((wpi * (rA[b, :n] * V[b, :n])).sum(1))
            F.append((wphi * (rA[b, :n] * U[b, :n])).sum(1))
        P, F = torch.stack(P), torch.stack(F)
        return P * P + F * F, P, F

    def residuals(self, U, V, A, d, m):
        q = U * U + V * V
        one = 1.0

        def D(e):
            return (e[:, :-4] - 8 * e[:, 1:-3] + 8 * e[:, 3:-1] - e[:, 4:]) / (12 * self.h)

        a1 = self.ext((A - one) * self.m1, 2, "eo")
        sc = torch.where(self.inner, self.sc, torch.ones_like(self.sc))
        rA = D(a1) - ((1 + 2 * self.s2) / sc * (1 - A) - sc * A * q)
        rd = D(self.ext(d, 2, "ee")) + sc * q
        E = torch.exp(-d)
        r0, r1, _, _ = self.rhs(U, V, A)
        qt = 2 * (U * r0 + V * r1)
        pt = self.sc * qt
        dt_ = -self.cell(pt, "oo") - self.h / 12 * pt[:, 1:2]
        Et = -E * dt_
        St = self.cell(self.t2 * (qt * E + q * Et), "ee")
        rt = -self.c3s * ((St - m * Et) / E) + 2 * self.sc * A * A * E * U * V
        z = torch.zeros_like(q)
        mx = lambda r: torch.where(self.inner, r.abs(), z).amax(1)  # noqa: E731
        M = self.cell(self.t2 * A * q, "ee").gather(1, self.n1)[:, 0]
        return torch.stack([mx(rA), mx(rd), mx(rt), m.gather(1, self.n1)[:, 0], M], 1)


def _seconds(case):
    """About how long `exact` takes: tensor operations times their time."""
    N = _grids(case)
    width = float(len(N) * N.max())
    op = max(9e-6, width * 8 * 3 / 3e12)
    if case["kind"] == "adjoint":
        return float(_n_steps(N.astype(np.float64), case["T"]).max()) * 4 * 300 * op * max(1, case["iters"]) * len(set(N))
    return case["steps"] * case["rk"] * 75 * op


def exact(case, seed):
    if _seconds(case) > 18.0:
        return None
    N = _grids(case)
    eps, sigma, c = _data(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    J = case["n_modes"]
    tabs = {int(n): [torch.from_numpy(a).to(dev) for a in _modes(int(n), max(J, 1))] for n in set(N.tolist())} if J else {}
    if case["kind"] == "adjoint":
        return _exact_gradient(case, N, eps, c, tabs, dev) if not case["iters"] else None
    X = _Exact(N, case, dev)
    V = torch.zeros_like(X.sc)
    for b, n in enumerate(N.tolist()):
        if c is None:
            t = np.tan((np.pi / 2) / (n - 1) * np.arange(n - 1))
            v = 2 * eps[b] / np.pi * np.exp(-4 * t * t / (np.pi * sigma[b]) ** 2)
            V[b, :n - 1] = torch.from_numpy(v).to(dev)
        else:
            V[b, :n - 1] = eps[b] * (torch.from_numpy(c[b]).to(dev) @ tabs[n][0][:case["coefs"]])[:-1]
    U = torch.zeros_like(V)
    rk, K = case["rk"], case["a_reint"]
    if case["kind"] in ("monitor", "analyse"):
        U, V, A = X.evolve(U, V, 64, rk, K)
        if case["kind"] == "monitor":
            U, V, A = X.evolve(U, V, case["steps"], rk, K)
        A, d, m = X.metric(U, V)
        res = X.residuals(U, V, A, d, m).cpu().numpy()
        if case["kind"] == "monitor":
            t = np.where(X.alive.cpu().numpy()[:, 0], case["steps"] * 0.25 * (math.pi / 2) / (N - 1), 0.0)
            if not bool(X.alive.all()):
                t = None
            return dict(status=dict(t=t, steps=None, state=None, t_c=None, minA=X.pack_min(A)), residuals=res)
        E, P, F = X.energies(U, V, A, tabs)
        return dict(E=E.cpu().numpy(), Pihat=P.cpu().numpy(), Phihat=F.cpu().numpy(), residuals=res)
    snaps = []

    def snap(n, U, V):
        snaps.append((U, V) + tuple(X.metric(U, V)))

    U, V, A = X.evolve(U, V, case["steps"], rk, K, snap if case["snap_every"] else None, case["snap_every"])
    if K and case["steps"] % K == 0:
        A = torch.where(X.alive, X.A_of(U * U + V * V), A)
    A, d, m = X.metric(U, V, A)
    fields = dict(Phi=U, Pi=V, A=A, delta=d, m=m)
    out = dict(status=dict(t=None, steps=None, state=None, t_c=None, minA=X.pack_min(A)),
               state={k: X.pack(v) for k, v in fields.items()})
    if snaps:
        out["snaps"] = torch.stack([torch.stack([X.pack(f) for f in s]) for s in snaps])
        if J:
            es = [X.energies(s[0], s[1], s[2], tabs) for s in snaps]
            out["spectra"] = tuple(torch.stack([e[k] for e in es]) for k in range(3))
        if len(snaps) != case["steps"] // case["snap_every"] + 1 or not bool(X.alive.all()):
            out["snaps"] = None
    return out


def _pack_min(self, A):
    one = torch.ones_like(A)
    return torch.minimum(torch.where(self.inner, A, one).amin(1), one[:, 0]).cpu().numpy()


_Exact.pack_min = _pack_min


def _exact_gradient(case, N, eps, c, tabs, dev):
    from torch.utils.checkpoint import checkpoint

    L, G = np.zeros(len(N)), np.zeros_like(c)
    for n in sorted(set(N.tolist())):
        at = np.flatnonzero(N == n)
        X = _Exact(N[at], case, dev)
        cc = torch.from_numpy(c[at]).to(dev).requires_grad_(True)
        e, wpi, wphi = tabs[n]
        V = torch.from_numpy(eps[at][:, None]).to(dev) * (cc @ e[:case["coefs"]]) * X.m1
        U = torch.zeros_like(V)

        def energies(U, V):
            rA = torch.sqrt(X.metric(U, V)[0])
            return ((rA * V) @ wpi[:16].T) ** 2 + ((rA * U) @ wphi[:16].T) ** 2

        E0 = energies(U, V)
        for _ in range(int(_n_steps(np.array([float(n)]), case["T"])[0])):
            U, V = checkpoint(lambda a, b: X.step4(a, b, X.dt)[:2], U, V, use_reentrant=False)
        l = ((energies(U, V) - E0) ** 2).sum(1)
        g, = torch.autograd.grad(l.sum(), cc)
        L[at], G[at] = l.detach().cpu().numpy(), g.cpu().numpy()
    return dict(L=L, dLdc=G, valid=None)
