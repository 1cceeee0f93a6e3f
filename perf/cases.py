"""Workloads the particle loop is timed on, over the range users run it in.

Three kinds of work, each through the public entry points of `paper_2107_07315_amd.sph`:

  steps      a run in progress: one `sph_step` call of several kick-drift-kick steps (with the
             candidate-list builds they need), the oscillation diagnostics recorded after it where
             the workload is an oscillation run; returns the whole state, the rates and the record.
  snapshot   one evaluation of a snapshot by a context that is kept: the arrays are loaded in the
             order they come in, then cells, density and EoS, stress rate, forces; returns every
             evaluated field.
  train      one epoch of the EoS network's training, with the holdout loss; returns the weights and
             the losses.

Workloads are those of `sph_inputs.workloads`.  A seed turns every star by a random rotation about its
centre and scales its velocities (the lattice draws its velocities), so another seed is another input
of the same physics; the placement itself is built once per size.  Runs with FP32 pair sums return
what a program stores of them: fields in float32, the precision of their sums, particles in the order of
their ids (rounding in FP32 can move a particle by one place in the framework's own order).
"""
import functools
import math

import numpy as np
import torch

from paper_2107_07315_amd import sph
from sph_inputs import eos_table as E
from sph_inputs import workloads as W

FIELDS = ("x", "y", "z", "vx", "vy", "vz", "u", "h", "S", "D", "rho", "P", "cs", "ax", "ay", "az", "dudt", "dSdt", "id")
RATES = ("D", "rho", "P", "cs", "ax", "ay", "az", "dudt", "dSdt", "id")
SKIN = {"FP64": 0.08, "FP32": 0.14}   # the binding's default Verlet skins (they decide when particles are re-sorted)
INPUTS = ("x", "y", "z", "vx", "vy", "vz", "u", "h", "S", "type", "broken", "id")


def listed():
    def steps(name, load, n, precision, k, **kw):
        return dict({"name": name, "kind": "steps", "load": load, "n": n, "precision": precision, "steps": k}, **kw)
    return [
        # the smallest run: the 16^3 periodic lattice of an elastic solid, its 10 steps in one call
        steps("lattice_4k_fp64", "lattice", 16 ** 3, "FP64", 10),
        # the paper's TOV-star oscillation run (about 15,000 particles), diagnostics every 10 steps
        steps("star_15k_fp64_diag", "star", 15_013, "FP64", 10, diag=True),
        # relaxing a star in the effective potential, with its wall and drag, before it is evolved
        steps("relax_20k_fp64", "relax", 20_000, "FP64", 10),
        # the Gamma = 2 star of the 100-step configuration
        steps("star_200k_fp64", "star", 200_003, "FP64", 10),
        # the 2M-particle tabulated-EoS star, plain FP64
        steps("ppstar_2m_fp64", "ppstar", 2_000_000, "FP64", 10),
        # the headline run: the same star with FP32 pair sums and the EoS network where it is trusted
        steps("ppstar_2m_fp32_net", "ppstar", 2_000_000, "FP32", 10, net=True),
        # the paper's crust shell: every particle stressed, walls at both faces, toroidal mode recorded
        steps("shell_1m_fp32_diag", "shell", 1_000_000, "FP32", 10, diag=True),
        # independent stars of uneven sizes in one particle set
        steps("ensemble_16_fp32", "ensemble", 1_000_003, "FP32", 10, stars=16),
        # first evaluation of a new star, as every run and every restart begins
        {"name": "snapshot_20k_fp64", "kind": "snapshot", "load": "star", "n": 19_997, "precision": "FP64"},
        {"name": "snapshot_300k_fp32", "kind": "snapshot", "load": "ppstar", "n": 300_007, "precision": "FP32"},
        {"name": "snapshot_1m_fp64", "kind": "snapshot", "load": "ppstar", "n": 1_000_003, "precision": "FP64"},
        # fitting the EoS network: one epoch over a million samples
        {"name": "train_1m", "kind": "train", "samples": 1_000_000, "epochs": 1, "batch": 4096},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(["steps"] * 6 + ["snapshot"] * 3 + ["train"])
    if kind == "train":
        return {"kind": "train", "samples": size(100_000, 1_000_000), "epochs": 1, "batch": 64 * rng.randint(16, 96)}
    precision = rng.choice(["FP64", "FP32"])
    if kind == "snapshot":
        return {"kind": "snapshot", "load": rng.choice(["star", "ppstar"]), "n": size(4_000, 1_000_000), "precision": precision}
    load = rng.choice(["lattice", "star", "star", "ppstar", "ppstar", "relax", "shell", "ensemble"])
    lo, hi = {"lattice": (8 ** 3, 64 ** 3), "star": (4_000, 1_000_000), "ppstar": (4_000, 2_000_000),
              "relax": (4_000, 60_000), "shell": (20_000, 300_000), "ensemble": (200_000, 1_000_000)}[load]
    case = {"kind": "steps", "load": load, "n": size(lo, hi), "precision": precision, "steps": 10}
    if load == "lattice":
        case["n"] = max(8, int(round(case["n"] ** (1.0 / 3.0)))) ** 3
    if load == "ensemble":
        case["stars"] = rng.randint(4, 16)
    if load in ("star", "shell"):
        case["diag"] = rng.random() < 0.5
    if load == "ppstar" and rng.random() < 0.5:
        case["net"] = True
    return case


# ---- inputs --------------------------------------------------------------------------------------


@functools.lru_cache(maxsize=3)
def _base(load, n, stars=0):
    """The workload at this size (placement, profile and parameters; seeds do not enter)."""
    if load == "lattice":
        return W.lattice(int(round(n ** (1.0 / 3.0))))
    if load == "star":
        return W.star(n)
    if load == "ppstar":
        return W.pp_star(n)
    if load == "relax":
        return W.relax_star(n)
    if load == "shell":
        return W.crust_shell(n)
    return W.ensemble(stars, n, nmin=max(1000, n // (4 * stars)), nmax=n, kind="pp")


def _inputs(case, seed):
    """(workload, arrays) of a case: the base workload, turned and perturbed by the seed."""
    w = _base(case["load"], case["n"], case.get("stars", 0))
    rng = np.random.Generator(np.random.PCG64(seed))
    a = w.copy_arrays()
    if case["load"] == "lattice":
        sigma = math.sqrt(float(np.mean(a["vx"] ** 2)))
        v = rng.normal(0.0, sigma, (3, w.n))
        v -= v.mean(axis=1, keepdims=True)
        a["vx"], a["vy"], a["vz"] = v
        return w, a
    if case["load"] == "shell":   # the imposed toroidal velocity of the oscillation run
        a["vx"], a["vy"], a["vz"] = (c.copy() for c in w.extra["v_tor"])
    groups = [(0, w.n, np.zeros(3))]
    if w.star_params is not None:
        off = w.star_offsets
        groups = [(int(off[s]), int(off[s + 1]), w.star_params[s, :3]) for s in range(len(w.star_params))]
    for lo, hi, centre in groups:
        q, r = np.linalg.qr(rng.normal(size=(3, 3)))
        q = q * np.sign(np.diag(r))
        scale = rng.uniform(0.8, 1.2)
        X = q @ np.stack([a[k][lo:hi] - c for k, c in zip("xyz", centre)])
        V = scale * (q @ np.stack([a[k][lo:hi] for k in ("vx", "vy", "vz")]))
        for k in range(3):
            a["xyz"[k]][lo:hi] = X[k] + centre[k]
            a[("vx", "vy", "vz")[k]][lo:hi] = V[k]
    return w, a


def _domain():
    """The EoS network's domain (the densest polytrope piece, a band around its cold curve): the box
    and the band's ln rho range and width."""
    pp = E.default_pp()
    band = E.piece_band(pp, 2, W.PP_RHOC, W.pp_table(), 0.045)
    return E.band_domain(pp, *band), band


@functools.lru_cache(maxsize=1)
def _network():
    """A network fitted outside the framework: seeded hidden layers, readout by least squares on the
    table (median error about 1e-5, so the 1e-4 trust mask accepts the band's interior).  Returns the
    hidden parameters and the readout in physical units."""
    dom, band = _domain()
    T = W.pp_table()
    rng = np.random.Generator(np.random.PCG64(1))

    def layer(nin):
        w = rng.normal(0.0, 1.0 if nin == 2 else 0.125, (64, nin)).astype(np.float32)
        if nin == 64:   # the values of BF16 weights
            bits = w.view(np.uint32)
            w = ((bits + 0x7FFF + ((bits >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32)
        return w, rng.uniform(-0.5, 0.5, 64).astype(np.float32)

    layers = [layer(2), layer(64), layer(64)]
    S = E.mlp_band_samples(E.default_pp(), *band, 20_000, 4)
    h = np.stack([(S[:, k] - dom[2 * k]) * 2.0 / (dom[2 * k + 1] - dom[2 * k]) - 1.0 for k in (0, 1)], axis=1)
    for w, b in layers:
        z = h @ w.T.astype(np.float64) + b
        h = z / (1.0 + np.exp(-z))
    fr, fu = (S[:, 0] - T.lnr0) / T.dlnr, (S[:, 1] - T.lnu0) / T.dlnu
    i, j = np.floor(fr).astype(int), np.floor(fu).astype(int)
    f, g = fr - i, fu - j
    t = np.stack([(1 - f) * ((1 - g) * A[i, j] + g * A[i, j + 1]) + f * ((1 - g) * A[i + 1, j] + g * A[i + 1, j + 1])
                  for A in (T.lnP, T.lncs2)], axis=1)
    sol = np.linalg.lstsq(np.concatenate([h, np.ones((len(h), 1))], axis=1), t, rcond=1e-6)[0]
    return [p.ravel() for wb in layers for p in wb], sol


def _load_network(ctx):
    hidden, sol = _network()
    ctx.mlp_set_domain(*_domain()[0])
    norm = ctx.mlp_get_norm().astype(np.float64)   # outputs: v = y scale + centre
    w4 = (sol[:64] / norm[6:8]).T.ravel()
    b4 = (sol[64] - norm[4:6]) / norm[6:8]
    ctx.mlp_set_params(np.concatenate(hidden + [w4, b4]).astype(np.float32))
    ctx.mlp_build_trust_mask(1e-4)


def _diag_params(w):
    """The radial band and the (r, theta) slab of the oscillation signals, by the star's or shell's size."""
    r = np.sqrt(w.arrays["x"] ** 2 + w.arrays["y"] ** 2 + w.arrays["z"] ** 2)
    R = float(r.max())
    return (0.4 * R, 0.6 * R, 0.5 * R, 0.1 * R, math.pi / 4, 0.2) if float(r.min()) < 0.5 * R else \
        (float(r.min()), R, 0.5 * (float(r.min()) + R), R, math.pi / 4, 0.2)


def prepare(case, seed):
    if case["kind"] == "train":
        dom, band = _domain()
        p = W.pp_star(4096).params.replace(eos="MLP")
        ctx = sph.Context(p, capacity=64)
        ctx.mlp_set_domain(*dom)
        ctx.mlp_set_params(E.mlp_init(seed % 1000 + 1))
        samples = torch.as_tensor(E.mlp_band_samples(E.default_pp(), *band, case["samples"], seed), device="cuda")
        return {"case": case, "ctx": ctx, "samples": samples}
    w, a = _inputs(case, seed)
    p = w.params.replace(precision=case["precision"])
    if case.get("net"):
        p = p.replace(eos="MLP")
    ctx = sph.Context(p, capacity=w.n)
    if w.star_params is not None:
        ctx.sph_ensemble_set(w.star_params)
    if case.get("net"):
        _load_network(ctx)
    st = sph.DeviceState(a)
    s = {"case": case, "ctx": ctx, "st": st, "dt": w.dt}
    if case["kind"] == "snapshot":
        s["source"] = {k: st[k].clone() for k in INPUTS}
        return s
    ctx.evaluate(st)
    if case["precision"] == "FP32":
        s["places"] = torch.arange(w.n, device="cuda")
    if case.get("diag"):
        s["diag"] = _diag_params(w)
        s["record"] = torch.zeros(10, dtype=torch.float64, device="cuda")
    return s


def _stored(st, places):
    """All fields in float32, particles by id: one (28, n) block."""
    at = torch.empty_like(places)
    at[st["id"].long()] = places
    rows = [st[k].view(-1, st.n) for k in FIELDS[:-1]]
    return torch.cat(rows).float().index_select(1, at)


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["kind"] == "train":
        hold = case["samples"] // 10
        hist = ctx.mlp_train(state["samples"], hold, case["epochs"], case["batch"], 1e-3)
        return {"params": ctx.mlp_get_params(), "history": hist}
    st = state["st"]
    if case["kind"] == "snapshot":
        for k, v in state["source"].items():
            st[k].copy_(v)
        ctx.evaluate(st)
        return {k: st[k].float() if case["precision"] == "FP32" and k != "id" else st[k] for k in RATES}
    ctx.sph_step(st, state["dt"], case["steps"])
    if case["precision"] == "FP32":
        block = _stored(st, state["places"])
        out = dict(zip(FIELDS[:8], block))
        out.update(S=block[8:14], dSdt=block[22:28], **dict(zip(FIELDS[9:17], block[14:22])))
    else:
        out = {k: st[k] for k in FIELDS}
    if "diag" in state:
        ctx.sph_diagnostics(st, *state["diag"], out=state["record"])
        rec = state["record"].float() if case["precision"] == "FP32" else state["record"]
        # kinetic, toroidal and internal energy, band mean of u, fit of v_theta; then the mode amplitude
        out["energies"], out["fit"], out["mode"] = rec[0:4], rec[4:7], rec[9:10]
    return out


def work(case):
    """Bytes: per evaluation and particle the 8 state values, type and broken flag read and the 8
    evaluated fields written (and the state written back where it is stepped); the stress and its rate
    for solids.  Flops: 32 per neighbour pair for the density and 63 for the forces, 300 a particle."""
    if case["kind"] == "train":
        done = (case["samples"] - case["samples"] // 10) // case["batch"] * case["batch"] * case["epochs"]
        fwd = 2.0 * (2 * 64 + 2 * 64 * 64 + 64 * 2)
        return {"bytes": 16.0 * case["samples"] + 8.0 * 8642, "flops": 3.0 * fwd * done + fwd * (case["samples"] // 10)}
    solid = 1.0 if case["load"] in ("lattice", "shell") else 0.0
    nb = {"lattice": 73.6, "star": 73.6, "shell": 60.0}.get(case["load"], 100.0)
    n, k = case["n"], case.get("steps", 1)
    per = 8 * 8 + 2 + 8 * 8 + (8 * 8 if case["kind"] == "steps" else 0) + solid * (3 if case["kind"] == "steps" else 2) * 48
    return {"bytes": float(n) * k * per, "flops": float(n) * k * (95.0 * nb + 300.0 + solid * 40.0 * nb)}


# ---- the same in plain 64-bit torch --------------------------------------------------------------


class _Reference:
    """The method in 64 bits, pair by pair: summation density, Gamma law or table, stress rate of solid
    particles, Monaghan viscosity, static isotropic background, external radial potential, and the
    kick-drift-kick step.  Results are reported in the framework's order, a Morton curve of 1024 cells an
    axis over the bounding box (equal keys in their previous order), taken again whenever a particle has
    moved plus grown by more than the skin since it was last taken."""

    def __init__(self, params, arrays, reach):
        self.p = params
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        f = {k: torch.as_tensor(np.asarray(arrays[k], np.float64), device=self.dev)
             for k in ("x", "y", "z", "vx", "vy", "vz", "u", "h")}
        self.X = torch.stack([f["x"], f["y"], f["z"]], 1)
        self.V = torch.stack([f["vx"], f["vy"], f["vz"]], 1)
        self.u, self.h = f["u"], f["h"]
        self.S = torch.as_tensor(np.asarray(arrays["S"], np.float64).T.copy(), device=self.dev)
        self.solid = torch.as_tensor(np.asarray(arrays["type"]) == 1, device=self.dev)
        self.id = torch.as_tensor(np.asarray(arrays["id"]), device=self.dev)
        self.S[~self.solid] = 0.0
        self.order = torch.arange(len(self.u), device=self.dev)
        self.reach, self.skin = reach, 0.0
        self._sort()
        self._find()

    def _sort(self):
        """The reporting order at the current positions."""
        p = self.p
        lo = torch.zeros(3, dtype=torch.float64, device=self.dev) if p.periodic else self.X.min(0).values
        ext = p.box if p.periodic else float((self.X.max(0).values - lo).max())
        g = ((self.X - lo) * (1024.0 / ext)).floor().clamp(0, 1023).to(torch.int64)
        key = torch.zeros(len(self.u), dtype=torch.int64, device=self.dev)
        for b in range(10):
            for d in range(3):
                key |= ((g[:, d] >> b) & 1) << (3 * b + d)
        self.order = self.order[torch.argsort(key[self.order], stable=True)]
        self.sorted_at = (self.X, self.h)

    def _find(self):
        self.pairs = self._pairs(self.reach)
        self.found_at = (self.X, self.h)

    def _moved(self, since):
        """Largest move plus growth since then, in smoothing lengths of then."""
        X, h = since
        return float(((self._wrap(self.X - X).norm(dim=1) + (self.h - h).clamp(min=0.0)) / h).max())

    def _wrap(self, d):
        if not self.p.periodic:
            return d
        return d - self.p.box * torch.round(d / self.p.box)

    def _pairs(self, reach):
        """Chunks (a, b) of ordered pairs with |x_a - x_b| < reach (h_a + h_b), a ascending: particles
        sorted along x, each chunk of targets against the window of x that can reach it."""
        n = len(self.u)
        xs, by = torch.sort(self.X[:, 0])
        Xs, hs = self.X[by], self.h[by]
        hmax = float(self.h.max())
        out, lo = [], 0
        while lo < n:
            hi = min(n, lo + max(64, 30_000_000 // max(1, n)))
            for _ in range(3):
                R = reach * (float(hs[lo:hi].max()) + hmax)
                if self.p.periodic:
                    w0, w1 = 0, n
                else:
                    w0 = int(torch.searchsorted(xs, xs[lo] - R))
                    w1 = int(torch.searchsorted(xs, xs[hi - 1] + R, right=True))
                grown = min(n, lo + max(64, 60_000_000 // max(1, w1 - w0)))
                if grown <= hi:
                    break
                hi = grown
            r2 = torch.zeros((hi - lo, w1 - w0), dtype=torch.float64, device=self.dev)
            for d in range(3):
                r2 += self._wrap(Xs[lo:hi, d, None] - Xs[None, w0:w1, d]) ** 2
            H = reach * (hs[lo:hi, None] + hs[None, w0:w1])
            a, b = torch.nonzero(r2 < H * H, as_tuple=True)
            a, b = by[a + lo], by[b + w0]
            keep = a != b
            out.append((a[keep], b[keep]))
            lo = hi
        return out

    def _metric(self, X):
        p = self.p
        rb = X.norm(dim=1)
        n = X / torch.where(rb > 0, rb, torch.ones_like(rb))[:, None]
        T = torch.as_tensor(np.asarray(p.bg_table, np.float64), device=self.dev)
        nb = T.shape[1]
        t = rb / p.bg_dr
        i = t.floor().clamp(0, nb - 2).to(torch.int64)
        f = t - i
        q = (1.0 - f) * T[:, i] + f * T[:, i + 1]
        a = p.bg_M / (2.0 * torch.where(rb > 0, rb, torch.ones_like(rb)))
        ext = torch.stack([(1 - a) / (1 + a), 2.0 / (1 + a) ** 2 * a / rb, 1 + a, -a / rb])
        q = torch.where(rb <= p.bg_dr * (nb - 1), q, ext)
        return q[0], q[1], q[2], q[3], n

    def _eos(self, rho, u):
        p = self.p
        if p.eos == "GAMMA_LAW":
            P = (p.gamma - 1.0) * rho * u
            return P, p.gamma * P / (rho * (1.0 + u + P / rho)) if p.background == "TOV" else p.gamma * P / rho
        T = p.table
        fr, fu = (rho.log() - T.lnr0) / T.dlnr, (u.log() - T.lnu0) / T.dlnu
        i = fr.floor().clamp(0, T.nr - 2).to(torch.int64)
        j = fu.floor().clamp(0, T.nu - 2).to(torch.int64)
        a, b = fr - i, fu - j
        out = []
        for A in (T.lnP, T.lncs2):
            A = torch.as_tensor(A, device=self.dev)
            out.append(((1 - a) * ((1 - b) * A[i, j] + b * A[i, j + 1]) + a * ((1 - b) * A[i + 1, j] + b * A[i + 1, j + 1])).exp())
        return out

    def _kernel(self, q, h):
        t = (1.0 - 0.5 * q).clamp(min=0.0)
        if self.p.kernel == "WC4":
            return (495.0 / (256.0 * math.pi) / h ** 3 * t ** 6 * (1 + 3 * q + 35.0 / 12.0 * q * q),
                    -1155.0 / (128.0 * math.pi) / h ** 5 * t ** 5 * (1 + 2.5 * q))
        return (21.0 / (16.0 * math.pi) / h ** 3 * t ** 4 * (1 + 2 * q), -105.0 / (16.0 * math.pi) / h ** 5 * t ** 3)

    def _each(self):
        """The neighbour pairs of the current positions: a, b, x_a - x_b, r^2, h_ab, W and F."""
        for a, b in self.pairs:
            d = self._wrap(self.X[a] - self.X[b])
            r2 = (d * d).sum(1)
            H = self.h[a] + self.h[b]
            k = r2 < H * H
            a, b, d, r2, hab = a[k], b[k], d[k], r2[k], 0.5 * H[k]
            yield (a, b, d, r2, hab) + self._kernel(r2.sqrt() / hab, hab)

    def evaluate(self):
        p, n = self.p, len(self.u)
        zero = lambda *s: torch.zeros((n,) + s, dtype=torch.float64, device=self.dev)   # noqa: E731
        D = self._kernel(zero(), self.h)[0]
        for a, b, d, r2, hab, Wk, F in self._each():
            D.index_add_(0, a, Wk)
        self.D = D = p.m * D
        tov = p.background == "TOV"
        v2 = (self.V * self.V).sum(1)
        if tov:
            al, dal, psi, dpsi, nr = self._metric(self.X)
            WL = 1.0 / (1.0 - psi ** 4 * v2 / al ** 2).sqrt()
            self.rho = D / (psi ** 6 * WL)
        else:
            self.rho = D.clone()
        self.P, cs2 = self._eos(self.rho, self.u)
        self.cs = cs2.sqrt()
        mu = torch.where(self.solid, p.mu_pfactor * self.P if p.mu_mode == "P_FACTOR" else torch.full_like(D, p.mu_const), 0.0)
        pi, sig = self.P / D ** 2, self.S / (D ** 2)[:, None]
        AP, AS, ud, G = zero(3), zero(3), zero(), zero(9)
        T6 = torch.tensor([0, 3, 4, 3, 1, 5, 4, 5, 2], device=self.dev)   # xx yy zz xy xz yz -> 3 x 3
        for a, b, d, r2, hab, Wk, F in self._each():
            v = self.V[a] - self.V[b]
            vr = (v * d).sum(1)
            m = hab * vr / (r2 + p.visc_eps * hab * hab)
            Pi = torch.where(vr < 0, (-p.visc_alpha * 0.5 * (self.cs[a] + self.cs[b]) * m + p.visc_beta * m * m)
                             / (0.5 * (D[a] + D[b])), 0.0)
            AP.index_add_(0, a, ((pi[a] + pi[b] + Pi) * F)[:, None] * d)
            ud.index_add_(0, a, (pi[a] + 0.5 * Pi) * F * vr)
            k = self.solid[a] | self.solid[b]
            a, b, d, v, F = a[k], b[k], d[k], v[k], F[k]
            s = (sig[a] + sig[b])[:, T6].view(-1, 3, 3)
            AS.index_add_(0, a, F[:, None] * (s @ d[:, :, None])[:, :, 0])
            G.index_add_(0, a, (-v[:, :, None] * (F[:, None] * d)[:, None, :]).reshape(-1, 9))
        AP, AS, ud, G = p.m * AP, p.m * AS, p.m * ud, p.m * G.view(-1, 3, 3)
        Gt = G.transpose(1, 2)
        e, R = (G + Gt) / (2 * D)[:, None, None], (G - Gt) / (2 * D)[:, None, None]
        S = self.S[:, T6].view(-1, 3, 3)
        tr = e.diagonal(dim1=1, dim2=2).sum(1) / 3.0
        dS = 2.0 * mu[:, None, None] * (e - tr[:, None, None] * torch.eye(3, dtype=torch.float64, device=self.dev)) + (R @ S - S @ R)
        dS = torch.where(self.solid[:, None, None], dS, 0.0)
        self.dS = torch.stack([dS[:, 0, 0], dS[:, 1, 1], dS[:, 2, 2], dS[:, 0, 1], dS[:, 0, 2], dS[:, 1, 2]], 1)
        sdot = torch.where(self.solid, (S * e).sum((1, 2)) / D, 0.0)
        if tov:
            hen = 1.0 + self.u + self.P / self.rho
            nv = (nr * self.V).sum(1)
            kP = al ** 2 * psi ** 2 / (WL * hen)
            B = (-((al * dal)[:, None] * nr + (4 * psi ** 3 * dpsi)[:, None] * (nv[:, None] * self.V - 0.5 * v2[:, None] * nr))
                 / (psi ** 4)[:, None] + (2 * dal / al * nv)[:, None] * self.V)
            self.A = -kP[:, None] * AP + B + AS
        else:
            self.A = -AP + AS
        if p.ext_table is not None:
            T = torch.as_tensor(np.asarray(p.ext_table, np.float64), device=self.dev)
            r = self.X.norm(dim=1)
            t = r / p.ext_dr
            i = t.floor().clamp(0, len(T) - 2).to(torch.int64)
            g = torch.where(t <= len(T) - 1, (1 - (t - i)) * T[i] + (t - i) * T[i + 1], 0.0)
            if p.wall_in > 0:
                g = g + p.wall_k * (p.wall_in - r).clamp(min=0.0)
            if p.wall_out > 0:
                g = g - p.wall_k * (r - p.wall_out).clamp(min=0.0)
            self.A = self.A + torch.where(r > 0, g / r, 0.0)[:, None] * self.X - p.damping * self.V
        self.du = ud + sdot

    def step(self, dt):
        p, hd = self.p, 0.5 * dt
        Vh, uh, Sh = self.V + hd * self.A, self.u + hd * self.du, self.S + hd * self.dS
        self.X = self.X + dt * Vh
        if p.periodic:
            self.X = torch.where(self.X >= p.box, self.X - p.box, torch.where(self.X < 0, self.X + p.box, self.X))
        self.V, self.u, self.S = Vh + hd * self.A, uh + hd * self.du, Sh + hd * self.dS
        if self._moved(self.sorted_at) > self.skin:
            self._sort()
        if self._moved(self.found_at) > self.reach - 1.0:
            self._find()
        self.evaluate()
        self.V, self.u, self.S = Vh + hd * self.A, uh + hd * self.du, Sh + hd * self.dS
        if p.h_mode == "ADAPTIVE":
            self.h = p.eta * (p.m / self.D) ** (1.0 / 3.0)

    def fields(self, names, by_id=False):
        f = dict(x=self.X[:, 0], y=self.X[:, 1], z=self.X[:, 2], vx=self.V[:, 0], vy=self.V[:, 1], vz=self.V[:, 2], u=self.u,
                 h=self.h, S=self.S, D=self.D, rho=self.rho, P=self.P, cs=self.cs, ax=self.A[:, 0], ay=self.A[:, 1],
                 az=self.A[:, 2], dudt=self.du, dSdt=self.dS)
        order = torch.argsort(self.id) if by_id else self.order
        return {k: f[k][order].T.contiguous() if k != "id" else None for k in names}

    def diagnostics(self, d):
        """Energies, band mean, fit of v_theta over the slab and l = 2 toroidal amplitude."""
        r_lo, r_hi, sr, dr, sth, dth = d
        X, V, m = self.X, self.V, self.p.m
        r, rc = X.norm(dim=1), X[:, :2].norm(dim=1)
        vphi = (X[:, 0] * V[:, 1] - X[:, 1] * V[:, 0]) / rc
        f = 3.0 * rc * X[:, 2] / r ** 2
        band = (r >= r_lo) & (r < r_hi)
        th = torch.acos(X[:, 2] / r)
        k = ((r - sr).abs() <= dr) & ((th - sth).abs() <= dth)
        vth = X[:, 2] / r * (X[:, 0] * V[:, 0] + X[:, 1] * V[:, 1]) / rc - rc / r * V[:, 2]
        A = torch.stack([torch.ones_like(r[k]), r[k] - sr, th[k] - sth], 1)
        fit = torch.linalg.solve(A.T @ A, A.T @ vth[k])
        one = torch.stack([0.5 * m * (V * V).sum(), 0.5 * m * (vphi * vphi).sum(), m * self.u.sum(), self.u[band].mean()])
        return {"energies": one, "fit": fit, "mode": ((vphi * f).sum() / (f * f).sum()).view(1)}


def exact(case, seed):
    """Plain 64-bit values for the Gamma-law and table runs up to 400k particles; none for the EoS network
    and its training (a fitted network has no 64-bit value of its own), ensembles, and runs whose pairs
    would take too long."""
    if case["kind"] == "train" or case.get("net") or case["load"] == "ensemble":
        return None
    if case["n"] > (1_100_000 if case["kind"] == "snapshot" else 250_000):
        return None
    w, a = _inputs(case, seed)
    if case["kind"] == "snapshot":
        ref = _Reference(w.params, a, 1.0)
        ref.evaluate()
        return ref.fields(RATES)
    if w.params.break_mode != "OFF" or w.params.y0_mode != "CONST":
        return None
    ref = _Reference(w.params, a, 1.2)
    ref.skin = SKIN[case["precision"]]
    ref.evaluate()
    for _ in range(case["steps"]):
        ref.step(w.dt)
    single = case["precision"] == "FP32"
    out = ref.fields(FIELDS[:-1] if single else FIELDS, by_id=single)
    if case.get("diag"):
        out.update(ref.diagnostics(_diag_params(w)))
    return out
