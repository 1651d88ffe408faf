"""Workloads the force loop is timed on, through the public ``md.Simulation`` calls.

Every case is what a user's program repeats: one force evaluation, or one
``step`` call of a run, with the energies or the mean square displacement read
afterwards where such a program reads them.  ``listed()`` names the sizes, each
with what it stands for; ``draw()`` gives others of the same ranges.  Inputs
are the package's own seeded systems; ``exact()`` repeats a case in plain FP64
PyTorch (pair lists by cell binning, knot sums term by term, the integrators
written out), with none of the package's arithmetic.

Keys of a case:
  system     bcc | fec | liquid | vacancy | piston | sheared
  mode       forces | nve | nvt | npt | gear
  cells      unit cells per edge (bcc, sheared, vacancy), or nx = ny (piston; nz)
  replicas   number of replicas (fec, liquid, vacancy)
  nmax       largest replica (fec: 250..nmax atoms, liquid: 128..nmax)
  potential, temperature, vacancies, skin, every (list rebuild period; 0 =
  automatic rebuilds), dt, precision, steps (per pass), graph (replay captured
  steps), sample (every k-th step's energies into the ring; 0 = none)
"""
import math
import random

import numpy as np
import torch

from paper_1107_2619_amd import inputs, md

DEVICE = "cuda:0"

DEFAULTS = {
    "system": "bcc", "mode": "nve", "cells": 10, "nz": 0, "replicas": 1, "nmax": 0, "potential": "fe_fs",
    "temperature": 300.0, "vacancies": 0.0, "skin": 0.3, "every": 10, "dt": 1.0, "precision": "fp64", "steps": 20,
    "graph": True, "sample": 0,
}


def _case(name, **kw):
    return {"name": name, **DEFAULTS, **kw}


def listed():
    return [
        # One force and energy evaluation of the smallest crystal the cutoff allows with
        # some room: what a minimiser or an outside integrator asks for at every move.
        _case("forces_250_fp64", mode="forces", cells=5, steps=1, graph=False),
        # The 2000-atom crystal of the paper's self-diffusion set-up: 100 steps, then the
        # energies are printed.  Launches and latency decide it.
        _case("bcc2000_fp64", cells=10, steps=100),
        # 25^3 cells, the size of the paper's comparison of lookup tables with direct
        # evaluation, with the 15-spline iron potential.
        _case("bcc31250_fe15_fp64", cells=25, potential="fe15_fs", skin=0.4, steps=40),
        # The headline: 1,013,760 atoms, 1% vacancies, 600 K, in both precisions.
        _case("bcc1m_fp64", cells=80, temperature=600.0, vacancies=0.01, skin=0.4),
        _case("bcc1m_mixed", cells=80, temperature=600.0, vacancies=0.01, skin=0.4, precision="mixed"),
        # Uneven Fe-C replicas in one batch (two species), 300-1200 K.
        _case("fec48_mixed", system="fec", replicas=48, nmax=16000, potential="fec_eam", skin=0.8, every=5,
              precision="mixed"),
        # Many small hot liquids, each rebuilt when its own atoms have moved far enough.
        _case("liquid256_auto_fp64", system="liquid", replicas=256, nmax=2000, temperature=2500.0, skin=0.5, every=0),
        # Self-diffusion: vacancy replicas at 900-2000 K under their thermostats, the mean
        # square displacement sampled after the steps.
        _case("vacancy192_nvt_mixed", system="vacancy", mode="nvt", cells=10, replicas=192, skin=0.5, every=5,
              precision="mixed"),
        # A shocked slab with a free axis and rigid atoms, the energies sampled on every step.
        _case("piston_fp64", system="piston", cells=30, nz=60, potential="cu_fs", dt=0.5, sample=1),
        # A crystal under hydrostatic pressure (its edges move).
        _case("npt16000_fp64", mode="npt", cells=20, temperature=600.0, skin=0.5),
        # The paper's other integrator.
        _case("gear54000_fp64", mode="gear", cells=30),
        # A sheared cell (edge vectors as columns).
        _case("sheared128k_mixed", system="sheared", cells=40, precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["forces", "bcc", "bcc", "fe15", "fec", "liquid", "vacancy", "piston", "npt", "gear", "sheared"])
    precision = rng.choice(["fp64", "mixed"])
    steps = rng.choice([20, 23, 40])
    if kind == "forces":
        c = _case("", mode="forces", cells=_log_int(rng, 4, 60), steps=1, graph=False)
    elif kind == "bcc":  # odd cell counts and vacancies: ragged sizes
        c = _case("", cells=_log_int(rng, 6, 62), temperature=float(rng.randint(200, 600)),
                  vacancies=round(rng.uniform(0.0, 0.02), 4), skin=0.4, steps=steps)
    elif kind == "fe15":
        c = _case("", cells=_log_int(rng, 8, 50), potential="fe15_fs", skin=0.4, steps=steps)
    elif kind == "fec":
        c = _case("", system="fec", replicas=_log_int(rng, 2, 24), nmax=_log_int(rng, 2000, 16000),
                  potential="fec_eam", skin=0.8, every=5, steps=steps)
    elif kind == "liquid":
        c = _case("", system="liquid", replicas=_log_int(rng, 4, 256), nmax=_log_int(rng, 300, 2000),
                  temperature=2500.0, skin=rng.choice([0.4, 0.5, 0.6]), every=0, steps=steps)
    elif kind == "vacancy":
        c = _case("", system="vacancy", mode="nvt", cells=rng.randint(6, 10), replicas=_log_int(rng, 2, 150), skin=0.5,
                  every=5, steps=steps)
    elif kind == "piston":
        c = _case("", system="piston", cells=rng.randint(6, 30), nz=rng.randint(12, 70), potential="cu_fs", dt=0.5,
                  sample=rng.choice([1, 5]), steps=steps)
    elif kind == "npt":
        c = _case("", mode="npt", cells=_log_int(rng, 8, 40), temperature=float(rng.randint(200, 600)), skin=0.5,
                  steps=steps)
    elif kind == "gear":
        c = _case("", mode="gear", cells=_log_int(rng, 6, 50), steps=steps)
    else:
        c = _case("", system="sheared", cells=_log_int(rng, 10, 45), steps=steps)
    c["precision"] = precision
    del c["name"]
    return c


# ----------------------------------------------------------------------------- inputs
SHEAR = np.array([[1.0, 0.0, 1.0], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0]])  # edge vectors of the sheared cell (the same crystal)
TAU_FS = 100.0  # thermostat period
PRESSURE_GPA = 2.0
BOX_MASS_PER_ATOM = 20.0  # eV fs^2 / A^2


def _system(c, seed):
    s = 1 + seed % 1_000_003
    common = {"dt_fs": c["dt"], "skin": c["skin"], "rebuild_every": max(c["every"], 1)}
    if c["system"] == "fec":
        # the sizes and carbon sites of the default seeds, velocities and potential of this one
        sys_ = inputs.fec_replicas(c["replicas"], 250, c["nmax"], pot_seed=s, **common)
        return _repeated(sys_, c["replicas"], s)
    if c["system"] == "vacancy":
        temps = [900 + 1100 * k / max(c["replicas"] - 1, 1) for k in range(c["replicas"])]
        return inputs.vacancy_replicas(temps, 1, c["cells"], seed0=s, pot_seed=s, **common)
    if c["system"] == "piston":
        return inputs.fcc_piston(c["cells"], c["cells"], c["nz"], seed=s, **common)
    if c["system"] == "liquid":
        # up to 16 packings, each run several times with velocities of its own
        # (equivalent runs, over which such a program averages); sizes of the default seeds
        n = min(16, c["replicas"])
        base = inputs.liquid_replicas(n, 128, c["nmax"], temperature=c["temperature"], pot_seed=s, **common)
        return _repeated(base, c["replicas"], s)
    return inputs.bcc_fe(c["cells"], temperature=c["temperature"], vacancy_frac=c["vacancies"], seed=s,
                         displace=0.05 if c["mode"] == "forces" else 0.0, potential=c["potential"], **common)


def _repeated(base, replicas, seed):
    rng = np.random.default_rng(seed)
    pick = np.arange(replicas) % base.n_replicas
    part = [slice(int(base.atom_offset[r]), int(base.atom_offset[r + 1])) for r in pick]
    mass = base.potential["mass"]
    vel = [inputs.maxwell_boltzmann(mass[base.species[p]], float(base.temperature[r]), rng) for r, p in zip(pick, part)]
    return inputs.System(
        name=base.name, pos=np.concatenate([base.pos[p] for p in part]), vel=np.concatenate(vel),
        species=np.concatenate([base.species[p] for p in part]), rigid=np.concatenate([base.rigid[p] for p in part]),
        atom_offset=np.concatenate([[0], np.cumsum([p.stop - p.start for p in part])]).astype(np.int64),
        box=base.box[pick], origin=base.origin[pick], periodic=base.periodic[pick],
        rigid_velocity=base.rigid_velocity[pick], potential=base.potential, dt_fs=base.dt_fs, skin=base.skin,
        rebuild_every=base.rebuild_every, steps=base.steps, temperature=base.temperature[pick],
        max_neighbours=base.max_neighbours,
    )


def _thermostat_mass(sys_):
    """Q = g k_B T tau^2 per replica (eV fs^2)."""
    n = np.diff(sys_.atom_offset)
    return (3 * n - 3) * KB_EV * sys_.temperature * TAU_FS * TAU_FS


def _box_matrix(sys_):
    return np.diag(sys_.box[0]) @ SHEAR


def prepare(case, seed):
    c = case
    sys_ = _system(c, seed)
    kw = {"precision": c["precision"]}
    if c["mode"] == "nvt":
        kw.update(nh_temperature=sys_.temperature, nh_mass=_thermostat_mass(sys_))
    if c["mode"] == "npt":
        kw.update(pr_pressure_gpa=[PRESSURE_GPA], pr_mass=[BOX_MASS_PER_ATOM * sys_.n_atoms])
    if c["mode"] == "gear":
        kw.update(integrator="gear3")
    if c["system"] == "sheared":
        kw.update(box_matrix=_box_matrix(sys_))
    if c["sample"]:
        kw.update(energy_ring=2 * c["steps"])
    sim = md.Simulation(sys_, device=DEVICE, **kw)
    if c["every"] == 0:
        sim.set_option(md.MD_OPT_AUTO_REBUILD, 1)
    if c["sample"]:
        sim.set_option(md.MD_OPT_ENERGY_EVERY, c["sample"])
    if c["graph"]:
        sim.set_option(md.MD_OPT_USE_GRAPH, 1)
    return {"case": c, "sim": sim}


def run(state):
    c, sim = state["case"], state["sim"]
    if c["mode"] == "forces":
        sim.eam_forces(want_energy=True)
    else:
        sim.step(c["steps"])
    out = {"f": (sim.fx, sim.fy, sim.fz), "e_atom": sim.e_atom}
    if c["mode"] != "forces":
        out.update(x=(sim.x, sim.y, sim.z), v=(sim.vx, sim.vy, sim.vz))
    if c["mode"] == "nvt":
        out["msd"] = sim.msd()[0]
    elif c["sample"]:
        h = sim.energy_history()
        out["history"] = np.array([np.concatenate([e.pe, e.ke, e.piston_work]) for e in h])
    elif c["mode"] in ("forces", "npt") or (c["system"] == "bcc" and c["mode"] == "nve"):
        e = sim.energy()
        out["energy"] = np.concatenate([e.pe, e.ke])
        out["virial"] = e.virial
        out["box"] = e.box
    return out


def _atoms(c):
    """(atoms, neighbours within the cutoff) of a case, without building it."""
    n = c["cells"]
    if c["system"] == "fec":
        return c["replicas"] * (250 + c["nmax"]) / 2, 26.0
    if c["system"] == "liquid":
        return c["replicas"] * (128 + c["nmax"]) / 2, 21.0
    if c["system"] == "piston":
        return 4 * n * n * c["nz"], 42.0
    return 2 * n**3 * (1 - c["vacancies"]) * c["replicas"], 26.0


def work(case):
    """One pass: every step reads and writes each atom's position and velocity (96
    bytes); the call writes forces and energies (32).  Each unordered pair within
    the cutoff takes its separation and distance twice (density, then force: 2 x 12),
    a density and two derivative cubics or quadratics (20) and both atoms' share (16)."""
    atoms, nbr = _atoms(case)
    if case["mode"] == "forces":
        return {"bytes": atoms * (24 + 32), "flops": atoms * (nbr / 2 * 60 + 20)}
    return {"bytes": atoms * (96 * case["steps"] + 32), "flops": atoms * case["steps"] * (nbr / 2 * 60 + 40)}


# ----------------------------------------------------------------------------- FP64 in plain PyTorch
KB_EV = 8.617343e-5
EV_J, AMU_KG = 1.60217653e-19, 1.66053886e-27
T0_FS = math.sqrt(AMU_KG * 1.0e-20 / EV_J) * 1.0e15  # sqrt(amu A^2 / eV)
GPA = 160.217653  # GPa per eV / A^3


class _Model:
    """Pairs, energies and forces of a batch of replicas in FP64."""

    def __init__(self, sys_, hmat):
        self.dev = torch.device(DEVICE if torch.cuda.is_available() else "cpu")
        t = lambda a: torch.as_tensor(np.asarray(a), device=self.dev)  # noqa: E731
        p = sys_.potential
        self.ns = len(p["mass"])
        flat = lambda a: t(a).reshape(self.ns * self.ns, -1)  # noqa: E731
        self.pa, self.pr, self.da, self.dr = (flat(p[k]) for k in ("pair_a", "pair_r", "dens_A", "dens_R"))
        self.c, self.mass = t(p["emb_c"]), t(p["mass"])
        self.rc = float(max(self.pr.max(), self.dr.max()))
        self.sp, self.rigid = t(sys_.species).long(), t(sys_.rigid).bool()
        self.off = [int(v) for v in sys_.atom_offset]
        self.n = self.off[-1]
        self.n_rep = len(self.off) - 1
        self.rep = torch.repeat_interleave(torch.arange(self.n_rep, device=self.dev), t(np.diff(sys_.atom_offset)))
        self.h = t(np.stack([np.diag(b) for b in sys_.box]) if hmat is None else hmat[None]).clone()
        self.o, self.per = t(sys_.origin), t(sys_.periodic).bool()
        self.m = self.mass[self.sp] * T0_FS * T0_FS  # eV fs^2 / A^2

    def list_pairs(self, x, margin):
        """Every directed pair closer than r_c + margin, with its image."""
        rl, got_i, got_j, got_s = self.rc + margin, [], [], []
        for r in range(self.n_rep):
            a, b = self.off[r], self.off[r + 1]
            h, hi = self.h[r], torch.linalg.inv(self.h[r])
            s = (x[a:b] - self.o[r]) @ hi.T
            per = self.per[r]
            img0 = torch.where(per, torch.floor(s), torch.zeros_like(s))
            s = s - img0
            width = 1.0 / torch.linalg.norm(hi, dim=1)
            nc = torch.clamp((width / rl).floor().long(), min=1)
            if bool((per & (nc < 3)).any()):
                i, j, sh = self._brute(s, h, per, rl)
            else:
                i, j, sh = self._binned(s, h, per, nc, rl)
            got_i.append(i + a)
            got_j.append(j + a)
            got_s.append(sh + img0[i] - img0[j])
        # one row of neighbours per atom, padded with the atom itself
        i, order = torch.sort(torch.cat(got_i), stable=True)
        count = torch.bincount(i, minlength=self.n)
        first = torch.cumsum(count, 0) - count
        at = (i, torch.arange(len(i), device=self.dev) - first[i])
        width = int(count.max())
        self.j = torch.arange(self.n, device=self.dev)[:, None].repeat(1, width)
        self.j[at] = torch.cat(got_j)[order]
        self.img = torch.zeros(self.n, width, 3, dtype=torch.float64, device=self.dev)
        self.img[at] = torch.cat(got_s)[order]
        self.live = torch.arange(width, device=self.dev)[None] < count[:, None]
        self.ab = self.sp[:, None] * self.ns + self.sp[self.j]
        self.ba = self.sp[self.j] * self.ns + self.sp[:, None]

    @staticmethod
    def _brute(s, h, per, rl):
        out = []
        for k in range(0, len(s), 1024):
            d = s[None] - s[k:k + 1024, None]
            n = torch.where(per, -torch.round(d), torch.zeros_like(d))
            r2 = (((d + n) @ h.T) ** 2).sum(-1)
            i, j = torch.nonzero(r2 < rl * rl, as_tuple=True)
            keep = i + k != j
            out.append((i[keep] + k, j[keep], n[i[keep], j[keep]]))
        return tuple(torch.cat(v) for v in zip(*out))

    @staticmethod
    def _binned(s, h, per, nc, rl):
        c = torch.minimum(torch.clamp((s * nc).floor().long(), min=0), nc - 1)
        key = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
        order = torch.argsort(key, stable=True)
        cells = int(nc.prod())
        count = torch.bincount(key, minlength=cells)
        start = torch.cumsum(count, 0) - count
        out = []
        for dz in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    cc = c + torch.tensor([dx, dy, dz], device=s.device)
                    wrap = torch.div(cc, nc, rounding_mode="floor")
                    ok = ((wrap == 0) | per).all(1)
                    cc = cc - wrap * nc
                    k = torch.where(ok, (cc[:, 2] * nc[1] + cc[:, 1]) * nc[0] + cc[:, 0], 0)
                    cnt = torch.where(ok, count[k], 0)
                    i = torch.repeat_interleave(torch.arange(len(s), device=s.device), cnt)
                    first = torch.cumsum(cnt, 0) - cnt
                    j = order[start[k][i] + torch.arange(len(i), device=s.device) - first[i]]
                    n = wrap[i].to(s.dtype)
                    r2 = (((s[j] - s[i] + n) @ h.T) ** 2).sum(1)
                    keep = (r2 < rl * rl) & (i != j)
                    out.append((i[keep], j[keep], n[keep]))
        return tuple(torch.cat(v) for v in zip(*out))

    def evaluate(self, x):
        """Forces, per-atom energies and the virial tensor [R, 6]."""
        d = x[self.j] - x[:, None]
        for b in range(3):
            d += self.img[:, :, b, None] * self.h[self.rep][:, None, :, b]
        r = torch.where(self.live, torch.sqrt((d * d).sum(2)), 2 * self.rc)  # padding: beyond every knot
        sums = lambda a, rk, ab, pw: sum(  # noqa: E731
            a[:, k][ab] * torch.clamp(rk[:, k][ab] - r, min=0.0) ** pw for k in range(a.shape[1]))
        rho = sums(self.da, self.dr, self.ab, 3).sum(1)
        c = self.c[self.sp]
        root = torch.sqrt(rho)
        emb = -c * root
        demb = torch.where(rho > 0, -0.5 * c / root, torch.zeros_like(rho))
        e = 0.5 * sums(self.pa, self.pr, self.ab, 3).sum(1) + emb
        g = -3 * (sums(self.pa, self.pr, self.ab, 2) + demb[:, None] * sums(self.da, self.dr, self.ab, 2)
                  + demb[self.j] * sums(self.da, self.dr, self.ba, 2))
        s = g / r
        f = (s[:, :, None] * d).sum(1)
        s = torch.where(self.rigid[:, None] & self.rigid[self.j], 0.0, s)
        w = [(s * d[:, :, a] * d[:, :, b]).sum(1) for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
        w = -0.5 * torch.stack([self.per_replica(v) for v in w], 1)
        return f, e, w

    def per_replica(self, v):
        return torch.stack([v[a:b].sum() for a, b in zip(self.off, self.off[1:])])

    def kinetic(self, v):
        return self.per_replica(torch.where(self.rigid, 0.0, 0.5 * self.m * (v * v).sum(1)))


def exact(case, seed):
    c = case
    if not torch.cuda.is_available() and _atoms(c)[0] * c["steps"] > 1e6:
        return None  # minutes without the GPU
    sys_ = _system(c, seed)
    M = _Model(sys_, _box_matrix(sys_) if c["system"] == "sheared" else None)
    t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=M.dev)  # noqa: E731
    x, v, x0 = t(sys_.pos), t(sys_.vel), t(sys_.pos)
    mob = (~M.rigid)[:, None]
    vp = t(sys_.rigid_velocity)[M.rep]
    im, dt = 1.0 / M.m[:, None], c["dt"]
    M.list_pairs(x, 0.0 if c["mode"] == "forces" else 0.8)
    f, e, w = M.evaluate(x)
    if c["mode"] == "forces":
        out = {"f": tuple(f.T), "e_atom": e}
        out["energy"] = torch.cat([M.per_replica(e), M.kinetic(v)])
        out["virial"], out["box"] = w, t(sys_.box)
        return out
    R = M.n_rep
    zero = torch.zeros(R, dtype=torch.float64, device=M.dev)
    pi, xi, work_, history = zero.clone(), zero.clone(), zero.clone(), []
    gkt = (3 * t(np.diff(sys_.atom_offset)) - 3) * KB_EV * t(sys_.temperature)
    Q = t(_thermostat_mass(sys_))
    L, Ld = t(sys_.box[0]), torch.zeros(3, dtype=torch.float64, device=M.dev)
    acc, jrk = f * im, torch.zeros_like(f)

    def thermostat(v, pi, xi):  # half a step
        hh, K = 0.5 * dt, M.kinetic(v)
        pi = pi + 0.5 * hh * (2 * K - gkt) / Q
        s = torch.exp(-pi * hh)
        xi = xi + pi * hh
        pi = pi + 0.5 * hh * (2 * K * s * s - gkt) / Q
        return v * s[M.rep][:, None], pi, xi

    def box_kick(v, L, Ld, w):  # half a step
        vol = L.prod()
        stress = ((M.m[:, None] * v * v).sum(0) + w[0, :3]) / vol
        return Ld + 0.5 * dt * (vol / L) * (stress - PRESSURE_GPA / GPA) / (BOX_MASS_PER_ATOM * M.n)

    def power(f):
        return M.per_replica(torch.where(M.rigid, -(f * vp).sum(1), 0.0))

    for k in range(1, c["steps"] + 1):
        if k % 5 == 0:
            M.list_pairs(x, 0.8)
        if c["mode"] == "gear":
            xp = x + v * dt + acc * (dt * dt / 2) + jrk * (dt**3 / 6)
            vq, ap = v + acc * dt + jrk * (dt * dt / 2), acc + jrk * dt
            f, e, w = M.evaluate(xp)
            d = (f * im - ap) * (dt * dt / 2)
            x, v = xp + d / 6, vq + (5 / 6) * d / dt
            acc, jrk = ap + d * (2 / (dt * dt)), jrk + (1 / 3) * d * (6 / dt**3)
            continue
        if c["mode"] == "nvt":
            v, pi, xi = thermostat(v, pi, xi)
        if c["mode"] == "npt":
            Ld = box_kick(v, L, Ld, w)
            v = v * torch.exp(-0.5 * dt * Ld / L)
        work_ = work_ + 0.5 * dt * power(f)
        v = torch.where(mob, v + 0.5 * dt * f * im, vp)
        if c["mode"] == "npt":
            u = dt * Ld / L
            phi = torch.where(u == 0, torch.ones_like(u), torch.log1p(u) / torch.where(u == 0, 1.0, u))
            grow = 1 + u
            x = x * grow + dt * phi * grow * v
            L = L * grow
            M.h = torch.diag(L)[None]
        else:
            x = x + dt * v
        f, e, w = M.evaluate(x)
        work_ = work_ + 0.5 * dt * power(f)
        v = torch.where(mob, v + 0.5 * dt * f * im, vp)
        if c["mode"] == "npt":
            v = v * torch.exp(-0.5 * dt * Ld / L)
            Ld = box_kick(v, L, Ld, w)
        if c["mode"] == "nvt":
            v, pi, xi = thermostat(v, pi, xi)
        if c["sample"] and k % c["sample"] == 0:
            history.append(torch.cat([M.per_replica(e), M.kinetic(v), work_]))
    out = {"f": tuple(f.T), "e_atom": e, "x": tuple(x.T), "v": tuple(v.T)}
    if c["mode"] == "nvt":
        n = t(np.diff(sys_.atom_offset))
        out["msd"] = (M.per_replica(((x - x0) ** 2).sum(1)) / n)[:, None]
    elif c["sample"]:
        out["history"] = torch.stack(history)
    elif c["mode"] == "npt" or (c["system"] == "bcc" and c["mode"] == "nve"):
        out["energy"] = torch.cat([M.per_replica(e), M.kinetic(v)])
        out["virial"], out["box"] = w, L[None]
    return out
