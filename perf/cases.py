"""Timed cases of the framework: what its users run, through its public entry
points, with seeded synthetic surveys in GPU memory.

Every case is a dict of plain values.  ``prepare`` builds what a program has in
hand before the call (velocities, density, wavelets, recorded data, the
``Survey`` or ``Inversion``), ``run`` makes one pass, ``exact`` computes the
same outputs in 64 bits with plain torch.

Kinds of case
  grad      one gradient of the misfit through ``BoreholeFWI`` (forward with
            checkpoints or the full velocity history, adjoint, finalize)
  forward   modelled traces only (observed data, trial steps of a line search)
  iterate   one ``Inversion`` iteration: with the parabolic line search, or the
            joint density inversion with the pseudo-Hessian and a radial taper
  picks     the starting model's stage: semblance, P and S picks, velocities
"""
from __future__ import annotations

import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_2005_00281_amd as P
from paper_2005_00281_amd import fwi

DEV = "cuda"
FLUID_VP, FLUID_RHO, HOLE = 1500.0, 1000.0, 0.1
TUNE_CACHE = os.path.join(os.path.dirname(os.path.abspath(P.__file__)), "tune_cache.json")

# Survey fields every wave case has: nshot, nr, nz (physical cells), pml, h (m),
# nt, f0 (Hz), ckpt (steps between checkpoints), nrec, order, hist ("ckpt" or
# "full"), ragged (shots of mixed sizes, each on its own stretch of the model),
# tuned (the shapes the tune cache holds for this survey).
_WAVE = dict(nshot=1, nr=128, nz=512, pml=20, h=5e-3, nt=1000, f0=10e3, ckpt=250, nrec=8,
             order=2, hist="ckpt", ragged=False, tuned=False, wavelet_grad=False)


def _wave(name, kind, **kw):
    c = dict(_WAVE, kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a unit-test sized model, latency of a whole gradient
        _wave("grad tiny", "grad", nr=24, nz=48, pml=6, nt=240, f0=40e3, ckpt=50, nrec=3),
        # a small single shot at its full record, checkpoints, the default tune
        _wave("grad 1x128x512", "grad", nt=4000),
        # the same tool position for source-signature estimation: the wavelet's
        # gradient too, and the full velocity history (it fits), odd sizes
        _wave("grad wavelet 1x163x709", "grad", nr=163, nz=709, nt=1501, hist="full",
              wavelet_grad=True),
        # one production shot at its full record with the shapes the tune cache
        # keeps for it (the recompute overlapped with the adjoint)
        _wave("grad 1x320x2048", "grad", nr=320, nz=2048, h=2.5e-3, nt=8000, f0=12e3, nrec=13,
              tuned=True),
        # a group of tool positions over one layered model, as the HBM planner
        # forms them; enough tiles to fill the chip
        _wave("grad 12x256x4096", "grad", nshot=12, nr=256, nz=4096, h=2.5e-3, nt=1250,
              nrec=13),
        # forward only: observed data or a line search's trial pass of that group
        _wave("forward 12x256x4096", "forward", nshot=12, nr=256, nz=4096, h=2.5e-3, nt=1250,
              nrec=13),
        # forward only of one ragged shot
        _wave("forward 1x301x1777", "forward", nr=301, nz=1777, h=2.5e-3, nt=1999, nrec=13),
        # one inversion iteration with the line search over shots of mixed size
        # and record length
        _wave("iterate ragged 6x384x3072", "iterate", nshot=6, nr=384, nz=3072, h=2.5e-3,
              nt=1400, nrec=13, ragged=True, mode="line_search"),
        # joint inversion of the moduli and the density
        _wave("iterate joint 1x160x768", "iterate", nr=160, nz=768, nt=1200, mode="joint"),
        # the fourth-order scheme on a small and on a production grid
        _wave("grad order4 1x128x512", "grad", nt=1000, order=4),
        _wave("grad order4 1x320x2048", "grad", nr=320, nz=2048, h=2.5e-3, nt=1000, nrec=13,
              order=4),
        # velocities for the starting model from the gathers of a survey
        dict(name="picks 64x13x16000", kind="picks", ngather=64, nrec=13, nt=16000, dt=0.25e-6,
             np=560, stride=10, win=600),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["grad", "grad", "grad", "forward", "forward", "iterate", "iterate",
                       "order4", "picks"])
    if kind == "picks":
        nt = int(_log(rng, 2000, 16000))
        win = rng.choice([200, 333, 600])
        return dict(kind="picks", ngather=int(_log(rng, 1, 64)), nrec=rng.choice([8, 13, 39]),
                    nt=nt, dt=0.25e-6, np=rng.randint(100, 560), stride=rng.choice([5, 10, 16]),
                    win=win)
    order = 4 if kind == "order4" else 2
    nr, nz = int(_log(rng, 48, 400)), int(_log(rng, 200, 6200))
    cells = (nr + 20) * (nz + 40)
    most = 2.0e9 if order == 4 else 1.0e10  # cell-steps of a pass's forward
    nt = int(_log(rng, 200, 4000))
    nt = max(200, min(nt, int(most / cells)))
    nshot = 1
    if order == 2 and rng.random() < 0.5:
        nshot = max(1, min(rng.randint(2, 16), int(most / (cells * nt)), int(16e6 / cells)))
    h = 2.5e-3 if nr >= 200 else 5e-3
    kw = dict(nshot=nshot, nr=nr, nz=nz, h=h, nt=nt, f0=float(int(rng.uniform(5e3, 20e3))),
              ckpt=rng.choice([100, 250, 250]), nrec=rng.choice([8, 13]), order=order,
              ragged=nshot > 1 and rng.random() < 0.5)
    if kind == "iterate":
        kw["mode"] = rng.choice(["line_search", "joint"])
    if kind == "grad":
        kw["wavelet_grad"] = rng.random() < 0.25
        if nshot == 1 and cells * nt < 6e9 and rng.random() < 0.4:
            kw["hist"] = "full"
    return _wave(None, "grad" if kind == "order4" else kind, **kw)


# ------------------------------------------------------------------- inputs
def _ricker(f0, dt, nt):
    a = (math.pi * f0 * ((np.arange(nt) + 0.5) * dt - 1.5 / f0)) ** 2
    return (1.0 - 2.0 * a) * np.exp(-a)


def _shots(c):
    """Geometry of each shot and the global grid (NRg, NZg)."""
    out, k0 = [], 0
    step = max(1, int(round(0.15 / c["h"])))
    p, h = c["pml"], c["h"]
    for s in range(c["nshot"]):
        nr, nz, nt = c["nr"], c["nz"], c["nt"]
        if c["ragged"]:  # mixed sizes and record lengths
            nr = max(32, nr * (3 - s % 3) // 3)
            nz = max(96, int(nz * (1.0 - 0.75 * ((s * 0.618) % 1.0))))
            nt = max(32, int(nt * (1.0 - 0.5 * ((s * 0.382) % 1.0))))
        T = nt * 1e-4 * h
        f0 = max(c["f0"], 3.0 / T)  # a short record takes a higher band
        zs = min(0.3, 0.2 * nz * h)
        last = 1.5 + 0.1524 * (c["nrec"] - 1)
        if last + 0.2 < nz * h and 1.2 / 4000.0 + 1.0 / f0 < T:
            # the tool's own spacing where the grid and the record hold it
            z = 1.5 + 0.1524 * np.arange(c["nrec"])
        else:  # an array that the record's waves reach
            far = max(2.5 * h * c["nrec"], min(0.7 * nz * h, 1600.0 * (T - 0.5 / f0)))
            z = zs + far * np.linspace(0.2, 1.0, c["nrec"])
        rec = p + np.floor(z / h + 0.5).astype(np.int32)
        out.append(SimpleNamespace(nr=nr, nz=nz, pr=p, pz=p, dr=h, dz=h, dt=1e-4 * h, nt=nt,
                                   f0=f0, vmax=5500.0, src_k=p + int(zs / h + 0.5),
                                   rec_k=rec, win_k0=k0, zs=zs, z=z))
        k0 += nz + 2 * p if c["ragged"] else step
    NZg = max(sh.win_k0 + sh.nz + 2 * p for sh in out)
    return out, max(sh.nr for sh in out) + p, NZg


def _earth(c, NR, NZ, seed):
    """Layered formation with a damaged zone around a water-filled hole, the
    velocities of an inversion under way: (vp, vs, rho) float32 arrays."""
    rng = np.random.default_rng([int(seed), 1])
    h, a = c["h"], min(HOLE, c["nr"] * c["h"] / 4)
    r = ((np.arange(NR) + 0.5) * h)[:, None]
    vp, vs, rho = (np.empty((NR, NZ), np.float32) for _ in range(3))
    k = 0
    while k < NZ:
        n = max(1, int(rng.uniform(0.2, 1.0) / h))
        v, q, d = rng.uniform(2500, 5400), rng.uniform(1.6, 2.0), rng.uniform(2100, 2700)
        depth, pct = rng.uniform(0.02, 0.3), rng.uniform(0.02, 0.25)
        f = 1.0 - pct * np.clip(1.0 - (r - a) / depth, 0.0, 1.0)
        vp[:, k:k + n], vs[:, k:k + n], rho[:, k:k + n] = v * f, v / q * f, d
        k += n
    fl = r[:, 0] < a
    vp[fl], vs[fl], rho[fl] = FLUID_VP, 0.0, FLUID_RHO
    return vp, vs, rho, fl


def _recorded(sh, wave, rng):
    """Recorded gather of a shot [nrec, nt]: direct fluid, P and S arrivals of
    the source's band with the amplitudes of a point source in water."""
    t = (np.arange(sh.nt) + 1.0) * sh.dt
    out = np.zeros((len(sh.z), sh.nt))
    for v, g in ((rng.uniform(3000, 5000), 0.3), (rng.uniform(1700, 2600), 0.6), (1450.0, 1.0)):
        for j, z in enumerate(sh.z):
            d = max(z - sh.zs, sh.dz)
            tau = t - d / v
            x = 2 * (math.pi * sh.f0) ** 2 * (tau - 1.5 / sh.f0)
            a = (math.pi * sh.f0 * (tau - 1.5 / sh.f0)) ** 2
            dw = np.where(tau > 0, x * (2 * a - 3) * np.exp(-a), 0.0)
            out[j] += g * dw / (4 * math.pi * FLUID_VP ** 2 * d)
    return out + 1e-3 * np.abs(out).max() * rng.standard_normal(out.shape)


def _host_inputs(c, seed):
    shots, NR, NZ = _shots(c)
    vp, vs, rho, fl = _earth(c, NR, NZ, seed)
    rng = np.random.default_rng([int(seed), 2])
    waves = [(_ricker(sh.f0, sh.dt, sh.nt) * rng.uniform(0.8, 1.2)).astype(np.float32)
             for sh in shots]
    obs = [_recorded(sh, w, rng).astype(np.float32) for sh, w in zip(shots, waves)]
    mask = np.zeros((NR, NZ), np.uint8)
    for sh in shots:
        mask[: sh.nr, sh.win_k0 + sh.pz: sh.win_k0 + sh.pz + sh.nz] = 1
    mask[fl] = 0
    return SimpleNamespace(shots=shots, NR=NR, NZ=NZ, vp=vp, vs=vs, rho=rho, waves=waves,
                           obs=obs, mask=mask)


def _gathers(c, seed):
    """Plane P and S arrivals in noise at a 13- (8-, 39-) receiver array."""
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    G, M, nt, dt = c["ngather"], c["nrec"], c["nt"], c["dt"]
    off = 0.1524 * torch.arange(M, device=DEV, dtype=torch.float32)
    t = torch.arange(nt, device=DEV, dtype=torch.float32) * dt
    vp = 3000 + 2500 * torch.rand(G, 1, 1, device=DEV, generator=g)
    ratio = 1.6 + 0.3 * torch.rand(G, 1, 1, device=DEV, generator=g)
    T = nt * dt

    def arrival(t0, p):
        a = (math.pi * 8e3 * (t - t0 - p * off[:, None])) ** 2
        return (1 - 2 * a) * torch.exp(-a)

    x = 3 * arrival(0.2 * T, 1 / vp) + arrival(0.45 * T, ratio / vp)
    x += 0.05 * torch.randn(x.shape, device=DEV, generator=g)
    return x, off.expand(G, M).contiguous()


def prepare(case, seed):
    c = case
    if c["kind"] == "picks":
        x, off = _gathers(c, seed)
        return SimpleNamespace(c=c, x=x, off=off)
    d = _host_inputs(c, seed)
    f32 = lambda a: torch.as_tensor(a, device=DEV)  # noqa: E731
    st = SimpleNamespace(c=c, vp=f32(d.vp), vs=f32(d.vs), rho=f32(d.rho))
    sv = P.Survey(d.shots, (d.NR, d.NZ), ckpt_every=min(c["ckpt"], c["nt"]), order=c["order"])
    st.sv, st.wav = sv, sv.pack_wavelets(d.waves)
    st.obs = f32(np.concatenate([o.ravel() for o in d.obs]))
    if c["tuned"]:
        lam, mu = P.moduli(st.vp, st.vs, st.rho)
        sv.autotune(lam, mu, st.rho, st.wav, cache=TUNE_CACHE)
    if c["hist"] == "full":
        sv.set_tune(full_history=1)
    if c["kind"] == "iterate":
        joint = c["mode"] == "joint"
        a = min(HOLE, c["nr"] * c["h"] / 4)
        taper = P.radial_taper(d.NR, c["h"], 0.5 * a, 1.5 * a) if joint else None
        st.inv = fwi.Inversion(sv, st.vp.clone(), st.vs.clone(), st.rho.clone(), st.wav, st.obs,
                               f32(d.mask), line_search=not joint, density=joint,
                               precond="pseudo_hessian" if joint else "illum",
                               row_weight=taper)
    return st


def run(state):
    st, c = state, state.c
    if c["kind"] == "picks":
        return _run_picks(st)
    if c["kind"] == "iterate":
        inv = st.inv
        inv.vp.copy_(st.vp)
        inv.vs.copy_(st.vs)
        inv.rho.copy_(st.rho)
        J, alpha = inv.iterate()
        out = {"J": J.float(), "alpha": alpha, "vp": inv.vp, "vs": inv.vs,
               "g_lam": inv.g_lam, "g_mu": inv.g_mu, "illum": inv.illum}
        if inv.density:
            out["rho"], out["g_rho"] = inv.rho, inv.g_rho
        return out
    if c["kind"] == "forward":
        lam, mu = P.moduli(st.vp, st.vs, st.rho)
        return {"traces": st.sv.fwd_model(lam, mu, st.rho, st.wav)}
    vp = st.vp.detach().requires_grad_(True)
    vs = st.vs.detach().requires_grad_(True)
    wav = st.wav.detach().requires_grad_(c["wavelet_grad"])
    lam, mu = P.Moduli.apply(vp, vs, st.rho)
    traces = P.BoreholeFWI.apply(lam, mu, st.sv, st.rho, wav)
    loss = 0.5 * ((traces - st.obs) ** 2).sum()
    loss.backward()
    out = {"traces": traces.detach(), "J": loss.detach(), "g_vp": vp.grad, "g_vs": vs.grad,
           "illum": st.sv.last_illum}
    if c["wavelet_grad"]:
        out["g_wavelet"] = wav.grad
    return out


P0, DP = 150e-6, 1e-6  # slowness scan, s/m


def _run_picks(st):
    c = st.c
    ntau = (c["nt"] - c["win"]) // c["stride"] + 1
    coh, en = P.semblance(st.x, c["dt"], st.off, P0, DP, c["np"], c["stride"], ntau, c["win"],
                          energy=True)
    pP, cP, proj = P.semblance_pick(coh, P0, DP, 1 / 6000, 1 / 2000, energy=en, rel_floor=1e-6,
                                    return_proj=True)
    pS, cS = P.semblance_pick(coh, P0, DP, 0.0, 0.999 / 1500, p_ref=pP, ref_scale=1.4,
                              energy=en, rel_floor=1e-6)
    return {"coh": coh, "energy": en, "proj": proj, "cP": cP, "cS": cS}


# --------------------------------------------------------------------- work
def work(case):
    c = case
    if c["kind"] == "picks":
        ntau = (c["nt"] - c["win"]) // c["stride"] + 1
        maps = c["ngather"] * c["np"] * ntau
        return {"bytes": 4.0 * (c["ngather"] * c["nrec"] * c["nt"] + 2 * maps),
                "flops": 6.0 * c["ngather"] * c["np"] * c["nrec"] * c["nt"]}
    shots, NR, NZ = _shots(c)
    steps = sum((sh.nr + sh.pr) * (sh.nz + 2 * sh.pz) * float(sh.nt) for sh in shots)
    cells, data = float(NR * NZ), float(sum(len(sh.z) * sh.nt for sh in shots))
    # operations per cell and step of the scheme as written: 46 forward, 85
    # adjoint with the correlation (order 4: 106 and 180)
    f, a = (46.0, 85.0) if c["order"] == 2 else (106.0, 180.0)
    if c["kind"] == "forward":
        return {"bytes": 4.0 * (3 * cells + data), "flops": f * steps}
    if c["kind"] == "grad":
        return {"bytes": 4.0 * (6 * cells + 2 * data), "flops": (f + a) * steps}
    joint = c["mode"] == "joint"
    return {"bytes": 4.0 * ((10 if joint else 8) * cells + data),
            "flops": (f + a + (20.0 if joint else f)) * steps}


# -------------------------------------------------------- the same in 64 bits
def _shift(x, d, axis, n=1):
    """x moved so that out[i] = x[i + n] along an axis (0 radial, 1 axial), zero outside."""
    if d == 0:
        return x
    out = torch.zeros_like(x)
    if axis == 0:
        if d > 0:
            out[:-d] = x[d:]
        else:
            out[-d:] = x[:d]
    elif d > 0:
        out[:, :-d] = x[:, d:]
    else:
        out[:, -d:] = x[:, :d]
    return out


class _Scheme:
    """The staggered velocity-stress step with CFS-PML in float64 torch."""

    def __init__(self, sh, order):
        self.sh, self.order = sh, order
        NR, NZ = sh.nr + sh.pr, sh.nz + 2 * sh.pz
        self.NR, self.NZ = NR, NZ
        D = dict(dtype=torch.float64, device=DEV)
        f = lambda x: float(np.float32(x))  # noqa: E731  the entry points take float32
        dr, dz, self.dt = f(sh.dr), f(sh.dz), f(sh.dt)
        self.dr, self.dz = dr, dz
        i = torch.arange(NR, **D)[:, None]
        self.rC, self.rR = (i + 0.5) * dr, i * dr
        self.rR[0] = 1.0
        self.up = (torch.arange(NR, device=DEV) >= 1).to(torch.float64)[:, None]

        def pml(x, n, hcell):
            if n == 0:
                return torch.zeros_like(x), torch.ones_like(x)
            d = -3.0 * f(sh.vmax) * math.log(1e-4) / (2.0 * n * hcell) * x * x
            al = math.pi * f(sh.f0) * (1.0 - x)
            b = torch.exp(-(d + al) * self.dt)
            a = d * (b - 1.0) / (d + al)
            on = x > 0
            return torch.where(on, a, 0.0 * a), torch.where(on, b, torch.ones_like(b))

        k = torch.arange(NZ, **D)[None, :]
        pen_r = lambda u: ((u - sh.nr) / max(1, sh.pr)).clamp(min=0.0)  # noqa: E731
        lo, hi = sh.pz - 0.5, sh.pz + sh.nz - 0.5
        pen_z = lambda u: (torch.maximum(lo - u, u - hi) / max(1, sh.pz)).clamp(min=0.0)  # noqa: E731
        self.ri, self.rh = pml(pen_r(i), sh.pr, dr), pml(pen_r(i + 0.5), sh.pr, dr)
        self.zi, self.zh = pml(pen_z(k), sh.pz, dz), pml(pen_z(k + 0.5), sh.pz, dz)
        scale = self.dt / (math.pi * dr * dr * dz)
        self.src = torch.zeros(NR, NZ, **D)
        self.src[0, sh.src_k] = scale * (math.sqrt(7.0 / 6.0) if order == 4 else 1.0)
        self.rec = torch.as_tensor(np.asarray(sh.rec_k, np.int64), device=DEV)

    def medium(self, lam, mu, rho):
        kp = lambda x: torch.cat([x[:, 1:], x[:, -1:]], 1)  # noqa: E731
        im = lambda x: torch.cat([x[:1], x[:-1]], 0)  # noqa: E731
        bR = self.up * 2.0 / (im(rho) + rho)
        bZ = 2.0 / (rho + kp(rho))
        four = (im(mu), mu, kp(im(mu)), kp(mu))
        solid = (four[0] > 0) & (four[1] > 0) & (four[2] > 0) & (four[3] > 0)
        inv = sum(1.0 / torch.where(solid, m, torch.ones_like(m)) for m in four)
        muS = self.up * torch.where(solid, 4.0 / inv, torch.zeros_like(mu))
        return self.dt * lam, 2.0 * self.dt * mu, self.dt * bR, self.dt * bZ, self.dt * muS

    # differences and averages from half to integer positions ("i": rows or
    # columns i-1 and i) and back ("h": i and i+1); across the axis fields at
    # half radial positions are even, those at integer ones odd
    def _four(self, x, axis, kind):
        d = (-1, 0, -2, 1) if kind == "i" else (0, 1, -1, 2)
        if axis == 1:
            return [_shift(x, q, 1) for q in d]
        if kind == "i":  # even field
            e = torch.cat([x[1:2], x[:1], x], 0)
        else:            # odd field, zero on the axis
            e = torch.cat([-x[2:3], -x[1:2], x], 0)
        e = torch.cat([e, torch.zeros_like(x[:2])], 0)
        n = x.shape[0]
        return [e[2 + q: 2 + q + n] for q in d]

    def diff(self, x, axis, kind):
        h = self.dr if axis == 0 else self.dz
        if self.order == 2:
            lo, hi = (-1, 0) if kind == "i" else (0, 1)
            return (_shift(x, hi, axis) - _shift(x, lo, axis)) / h
        m, p, mm, pp = self._four(x, axis, kind)
        return (9.0 / 8.0 * (p - m) - (pp - mm) / 24.0) / h

    def mean(self, x, kind):
        if self.order == 2:
            lo, hi = (-1, 0) if kind == "i" else (0, 1)
            return 0.5 * (_shift(x, hi, 0) + _shift(x, lo, 0))
        m, p, mm, pp = self._four(x, 0, kind)
        return 9.0 / 16.0 * (p + m) - (pp + mm) / 16.0

    def zero(self):
        return [torch.zeros(self.NR, self.NZ, dtype=torch.float64, device=DEV)
                for _ in range(14)]

    def step(self, s, med, w):
        cl, c2m, bR, bZ, mS = med
        vr, vz, trr, ttt, tzz, trz, A, B, C, D, E, F, G, H = s
        up = self.up

        def damp(psi, d, ab):
            psi = ab[1] * psi + ab[0] * d
            return psi, d + psi

        A, dr_ = damp(A, self.diff(trr, 0, "i"), self.ri)
        B, dz_ = damp(B, self.diff(trz, 1, "i"), self.zi)
        vr = vr + bR * (dr_ + dz_ + self.mean(trr - ttt, "i") / self.rR)
        C, dr_ = damp(C, self.diff(trz, 0, "h"), self.rh)
        D, dz_ = damp(D, self.diff(tzz, 1, "h"), self.zh)
        vz = vz + bZ * (dr_ + dz_ + self.mean(trz, "h") / self.rC)
        e = self.rates(vr, vz)
        E, err = damp(E, e[0], self.rh)
        F, ezz = damp(F, e[2], self.zi)
        G, ez = damp(G, e[3], self.zh)
        H, er = damp(H, e[4], self.ri)
        p = cl * (err + e[1] + ezz) + self.src * w
        trr = trr + p + c2m * err
        ttt = ttt + p + c2m * e[1]
        tzz = tzz + p + c2m * ezz
        trz = trz + mS * (ez + er)
        return [vr, vz, trr, ttt, tzz, trz, A, B, C, D, E, F, G, H * up]

    def rates(self, vr, vz):
        return (self.diff(vr, 0, "h"), self.mean(vr, "h") / self.rC, self.diff(vz, 1, "i"),
                self.diff(vr, 1, "h"), self.diff(vz, 0, "i"))

    def trace(self, s):
        return (s[2][0, self.rec] + s[3][0, self.rec] + s[4][0, self.rec]) / 3.0


def _exact_shot(sh, order, lam, mu, rho, wave, obs, want_grad, hessian=False):
    """Traces and, with want_grad, the gradients of 0.5 sum (traces - obs)^2 with
    respect to (lam, mu, rho, wave), the illumination and the pseudo-Hessian."""
    S = _Scheme(sh, order)
    seg = 40
    r = SimpleNamespace(illum=0.0, hl=0.0, hm=0.0)
    keep, tr = [], []
    with torch.no_grad():
        med, s = S.medium(lam, mu, rho), S.zero()
        for n in range(sh.nt):
            if n % seg == 0:
                keep.append(s)
            s = S.step(s, med, wave[n])
            tr.append(S.trace(s))
            if want_grad:
                vr, vz = s[0], s[1]
                ur, uz = vr + _shift(vr, 1, 0), vz + _shift(vz, -1, 1)
                r.illum = r.illum + 0.25 * S.dt * (ur * ur + uz * uz)
                if hessian:
                    e = S.rates(vr, vz)
                    es = S.up * (e[3] + e[4])
                    r.hl = r.hl + 3 * S.dt ** 2 * (e[0] + e[1] + e[2]) ** 2
                    r.hm = r.hm + S.dt ** 2 * (4 * (e[0] ** 2 + e[1] ** 2 + e[2] ** 2) + es * es)
    r.traces = torch.stack(tr, 1)
    if not want_grad:
        return r
    res = r.traces - obs
    r.J = 0.5 * float((res * res).sum())
    mdl = [x.detach().requires_grad_(True) for x in (lam, mu, rho)]
    med = S.medium(*mdl)
    cut = [m.detach().requires_grad_(True) for m in med]
    g_med = [torch.zeros_like(m) for m in cut]
    g_w = torch.zeros_like(wave)
    adj = None
    for j in range(len(keep) - 1, -1, -1):
        n0, n1 = j * seg, min(sh.nt, (j + 1) * seg)
        s0 = [x.detach().requires_grad_(True) for x in keep[j]]
        keep[j] = None
        w = wave[n0:n1].detach().requires_grad_(True)
        s, L = s0, 0.0
        for n in range(n0, n1):
            s = S.step(s, cut, w[n - n0])
            L = L + (S.trace(s) * res[:, n]).sum()
        if adj is not None:
            L = L + sum((x * a).sum() for x, a in zip(s, adj))
        g = torch.autograd.grad(L, s0 + cut + [w], allow_unused=True)
        adj = [torch.zeros_like(x) if y is None else y for x, y in zip(s0, g[:14])]
        for q in range(5):
            g_med[q] += g[14 + q]
        g_w[n0:n1] = g[19]
    r.g_lam, r.g_mu, r.g_rho = torch.autograd.grad(
        sum((m * g).sum() for m, g in zip(med, g_med)), mdl)
    r.g_w = g_w
    return r


def _exact_all(d, order, lam, mu, rho, want_grad, hessian=False):
    """Every shot of the survey, the gradients summed over their windows."""
    out = SimpleNamespace(traces=[], g_w=[], J=0.0)
    names = ("g_lam", "g_mu", "g_rho", "illum") + (("hl", "hm") if hessian else ())
    for n in names:
        setattr(out, n, torch.zeros_like(lam))
    for sh, w, o in zip(d.shots, d.waves, d.obs):
        win = (slice(0, sh.nr + sh.pr), slice(sh.win_k0, sh.win_k0 + sh.nz + 2 * sh.pz))
        r = _exact_shot(sh, order, lam[win], mu[win], rho[win],
                        torch.as_tensor(w, device=DEV).double(),
                        torch.as_tensor(o, device=DEV).double(), want_grad, hessian)
        out.traces.append(r.traces.reshape(-1))
        if want_grad:
            out.g_w.append(r.g_w)
            out.J += r.J
            for n in names:
                getattr(out, n)[win] += getattr(r, n)
    out.traces = torch.cat(out.traces)
    if want_grad:
        out.g_w = torch.cat(out.g_w)
    return out


def _exact_seconds(c):
    """About how long exact() takes."""
    shots, _, _ = _shots(c)
    t = 0.0
    for sh in shots:
        cells = (sh.nr + sh.pr) * (sh.nz + 2 * sh.pz)
        one = max(6e-4, 1.6e-9 * cells) * (1.6 if c["order"] == 4 else 1.0)
        t += sh.nt * one * {"forward": 1.0, "grad": 5.0, "iterate": 6.0}[c["kind"]]
    return t


def exact(case, seed):
    c = case
    if c["kind"] == "picks":
        return _exact_picks(c, seed)
    if _exact_seconds(c) > 13.0:
        return None
    d = _host_inputs(c, seed)
    f64 = lambda a: torch.as_tensor(a, device=DEV).double()  # noqa: E731
    vp, vs, rho = f64(d.vp), f64(d.vs), f64(d.rho)
    mu = rho * vs * vs
    lam = rho * vp * vp - 2.0 * mu
    if c["kind"] == "forward":
        return {"traces": _exact_all(d, c["order"], lam, mu, rho, False).traces}
    if c["kind"] == "iterate":
        return _exact_iterate(c, d, lam, mu, rho)
    r = _exact_all(d, c["order"], lam, mu, rho, True)
    out = {"traces": r.traces, "J": torch.tensor(r.J, dtype=torch.float64),
           "g_vp": 2 * rho * vp * r.g_lam, "g_vs": 2 * rho * vs * (r.g_mu - 2 * r.g_lam),
           "illum": r.illum}
    if c["wavelet_grad"]:
        out["g_wavelet"] = r.g_w
    return out


def _exact_iterate(c, d, lam, mu, rho):
    """Inversion.iterate with its default step (eps 1e-3, eta 0.02) and bounds."""
    joint = c["mode"] == "joint"
    m = torch.as_tensor(d.mask, device=DEV).bool()
    eps, eta = 1e-3, 0.02
    vp0, vp1, vs0, vs1 = 1000.0, 7000.0, 300.0, 4500.0
    r = _exact_all(d, c["order"], lam, mu, rho, True, hessian=joint)
    top = lambda x: float(x[m].abs().max())  # noqa: E731
    out = {"J": torch.tensor(r.J, dtype=torch.float64), "illum": r.illum}

    def scaled(g, diag, w):
        return torch.where(m, g * w / (diag + eps * float(diag[m].max())), 0.0 * g)

    w = 1.0
    if joint:
        a = min(HOLE, c["nr"] * c["h"] / 4)
        rr = (torch.arange(d.NR, device=DEV, dtype=torch.float64)[:, None] + 0.5) * c["h"]
        w = torch.sin(0.5 * math.pi * ((rr - 0.5 * a) / a).clamp(0, 1)) ** 2
        g = scaled(r.g_rho, r.illum, w)
        al = eta * top(rho) / top(g) if top(g) > 0 else 0.0
        rho = torch.where(m, (rho - al * g).clamp(1000.0, 3500.0), rho)
        out["rho"], out["g_rho"] = rho, g
    dl, dm = (r.hl, r.hm) if joint else (r.illum, r.illum)
    gl, gm = scaled(r.g_lam, dl, w), scaled(r.g_mu, dm, w)
    ratio = max(top(gl) / top(lam), top(gm) / top(mu))
    alpha = eta / ratio if ratio > 0 else 0.0

    def moved(al):
        mu1 = (mu - al * gm).clamp(min=rho * vs0 ** 2, max=rho * vs1 ** 2)
        p = (lam - al * gl + 2 * mu1).clamp(min=rho * vp0 ** 2, max=rho * vp1 ** 2)
        return torch.where(m, p - 2 * mu1, lam), torch.where(m, mu1, mu)

    if not joint:
        gpg = float((r.g_lam * gl)[m].sum() + (r.g_mu * gm)[m].sum())
        l1, m1 = moved(alpha)
        t1 = _exact_all(d, c["order"], l1, m1, rho, False).traces
        obs = torch.as_tensor(np.concatenate([o.ravel() for o in d.obs]), device=DEV).double()
        J1 = 0.5 * float(((t1 - obs) ** 2).sum())
        curv = (J1 - r.J + gpg * alpha) / alpha ** 2
        if curv > 0:
            alpha = min(max(gpg / (2 * curv), 0.1 * alpha), 3.0 * alpha)
        elif J1 > r.J:
            alpha *= 0.5
    lam, mu = moved(alpha)
    out.update(alpha=torch.tensor(alpha, dtype=torch.float64), g_lam=gl, g_mu=gm,
               vp=torch.sqrt((lam + 2 * mu) / rho), vs=torch.sqrt(mu / rho))
    return out


def _exact_picks(c, seed):
    x, off = _gathers(c, seed)
    G, M, nt = x.shape
    npp, stride, win = c["np"], c["stride"], c["win"]
    ntau = (nt - win) // stride + 1
    f = lambda v: float(np.float32(v))  # noqa: E731
    p0, dp, dt = f(P0), f(DP), f(c["dt"])
    starts = torch.arange(ntau, device=DEV) * stride
    n = torch.arange(nt, device=DEV)
    coh = torch.empty(G, npp, ntau, dtype=torch.float64, device=DEV)
    en = torch.empty_like(coh)
    offs = off[0].double().cpu().numpy()
    xd = torch.nn.functional.pad(x.double(), (0, 1))
    for j in range(npp):
        stack = torch.zeros(G, nt, dtype=torch.float64, device=DEV)
        power = torch.zeros_like(stack)
        for q in range(M):
            s = (p0 + j * dp) * float(offs[q]) / dt
            fl = math.floor(s)
            fr = s - fl
            at = n + int(fl)
            ok = (at >= 0) & ((at < nt - 1) | ((at == nt - 1) & (fr == 0.0)))
            ai = at.clamp(0, nt - 1)
            a, b = xd[:, q][:, ai], xd[:, q][:, ai + 1]
            v = torch.where(ok, a + fr * (b - a), 0.0 * a)
            stack += v
            power += v * v
        cs = torch.nn.functional.pad((stack * stack).cumsum(1), (1, 0))
        ce = torch.nn.functional.pad(power.cumsum(1), (1, 0))
        num, den = cs[:, starts + win] - cs[:, starts], ce[:, starts + win] - ce[:, starts]
        coh[:, j], en[:, j] = torch.where(den > 0, num / (M * den), 0.0 * num), den
    return {"coh": coh, "energy": en, "proj": None, "cP": None, "cS": None}
