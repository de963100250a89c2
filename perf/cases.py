"""Timed cases of the framework's main paths, with an independent FP64 answer.

A case is a dict of plain values; `listed()` names the standing ones, `draw`
gives further ones of the same ranges.  `prepare` makes what a program holds
before the call (a Sim with its particles loaded, saved states, output
arrays), `run` is one pass through the public entry points, `work` the bytes
and operations that pass cannot do without, `exact` the same pass in plain
torch FP64 without any of the framework's code.

Kinds of case:
  tick     one step of a small plasma, the inner loop of an interactive run
           (launches and latency count); also the plain FP64 path
  steps    a periodic FP32 run resumed from a saved state: K steps with the
           configured sorting, then a dump of fields and particles
  box      the same for the laser-wakefield box: walls, laser sheet,
           per-particle weights
  window   the two-dimensional wakefield run: moving window, injection,
           forced sorts, thin-grid tiles
  adjoint  a differentiable run: forward with checkpoints, then gradients
  guide    the waveguide of the field solver's convergence table, no particles
  monitor  a step followed by the full diagnostics

Particles are returned by their ids (storage order is the framework's own
business); positions as the displacement from the start of the pass's inputs,
wrapped to the box, so that a particle next to a periodic face reads the same
on both sides of it.
"""
from __future__ import annotations

import ctypes as C
import math

import numpy as np
import torch

PERIODIC, ABSORBING, PEC = 0, 1, 2
M_PROTON = 1836.0
DEV = "cuda"


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # The smallest FP32 step: the 16^3 thermal Langmuir plasma, one step per
        # call as a script that looks at its fields after every step makes them.
        {"name": "tick_f32_16", "kind": "tick", "nx": 16, "ny": 16, "nz": 16, "ppc": 8,
         "plasma": "langmuir", "precision": "fp32", "sort": -1, "steps": 1},
        # The plain FP64 path, two species: reference runs of a small box.
        {"name": "tick_f64_64", "kind": "tick", "nx": 64, "ny": 64, "nz": 64, "ppc": 8,
         "plasma": "thermal", "precision": "fp64", "sort": 0, "steps": 2},
        # A ragged grid (no side a multiple of a tile's), few particles per
        # cell, with the current filter of a smoothed run.
        {"name": "ragged_filter", "kind": "steps", "nx": 75, "ny": 49, "nz": 53, "ppc": 4,
         "plasma": "thermal", "order": 1, "passes": 1, "comp": 1, "sort": 10, "steps": 20},
        # The benchmark plasma: electrons and protons, 128^3, adaptive sorting,
        # over one of its sorting periods.
        {"name": "thermal_128", "kind": "steps", "nx": 128, "ny": 128, "nz": 128, "ppc": 8,
         "plasma": "thermal", "order": 1, "passes": 0, "comp": 0, "sort": -1, "steps": 30},
        # The largest: the hot anisotropic plasma, 268 M particles, most of
        # them crossing a cell face in every step, sorted every 10 steps.
        {"name": "anisotropic_256", "kind": "steps", "nx": 256, "ny": 256, "nz": 256, "ppc": 16,
         "plasma": "anisotropic", "order": 1, "passes": 0, "comp": 0, "sort": 10, "steps": 20},
        # Second-order shapes on the benchmark plasma.
        {"name": "order2_128", "kind": "steps", "nx": 128, "ny": 128, "nz": 128, "ppc": 8,
         "plasma": "thermal", "order": 2, "passes": 0, "comp": 0, "sort": -1, "steps": 8},
        # The wakefield box with a pulse inside: few particles per cell, so the
        # grid's work weighs as much as the particles'.
        {"name": "box_1024", "kind": "box", "nx": 1024, "ny": 128, "nz": 128, "ppc": 2,
         "sort": -1, "steps": 10},
        # The two-dimensional wakefield run at its largest particle count; two
        # window shifts and their sorts fall into a pass.
        {"name": "window_ppc32", "kind": "window", "nx": 1400, "nz": 300, "ppc": 32, "sort": -1,
         "steps": 32},
        # The differentiable run at its configured 32^3 (launches count).
        {"name": "adjoint_32", "kind": "adjoint", "nx": 32, "ny": 32, "nz": 32, "ppc": 16,
         "plasma": "cold", "sorted": False, "steps": 20, "every": 10},
        # The differentiable run at 33.5 M particles, sorted at its checkpoints.
        {"name": "adjoint_128", "kind": "adjoint", "nx": 128, "ny": 128, "nz": 128, "ppc": 16,
         "plasma": "anisotropic", "sorted": True, "steps": 10, "every": 5},
        # The field solver alone: the waveguide's fourth mesh (odd sizes, walls,
        # port, absorbing end).
        {"name": "guide_91x46x3001", "kind": "guide", "nx": 91, "ny": 46, "nz": 3001,
         "steps": 50},
        # A run that writes its energies and charge checks after every step.
        {"name": "monitor_128", "kind": "monitor", "nx": 128, "ny": 128, "nz": 128, "ppc": 8,
         "plasma": "thermal", "order": 1, "sort": -1, "steps": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tick", "tick", "steps", "steps", "steps", "box", "window", "adjoint",
                       "guide", "monitor"])
    if kind == "tick":
        prec = rng.choice(["fp32", "fp64"])
        hi = 40 if prec == "fp32" else 80
        nx, ny, nz = (_log_int(rng, 8, hi) for _ in range(3))
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "ppc": rng.choice([2, 4, 8, 16]),
                "plasma": rng.choice(["langmuir", "thermal"]), "precision": prec,
                "sort": -1 if prec == "fp32" else 0, "steps": rng.choice([1, 2, 4])}
    if kind == "steps":
        order = rng.choice([1, 1, 1, 2])
        nx, ny, nz = (_log_int(rng, 16, 160) for _ in range(3))
        passes = rng.choice([0, 0, 0, 1, 2])
        ppc = rng.choice([p for p in (1, 2, 4, 8, 16, 32) if nx * ny * nz * p <= 40_000_000])
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "ppc": ppc,
                "plasma": rng.choice(["thermal", "anisotropic"]), "order": order,
                "passes": passes, "comp": rng.choice([0, 1]) if passes else 0,
                "sort": rng.choice([-1, 5, 10]), "steps": rng.randint(6, 24) if order == 1 else 6}
    if kind == "box":
        return {"kind": kind, "nx": _log_int(rng, 128, 1100), "ny": _log_int(rng, 24, 128),
                "nz": _log_int(rng, 24, 128), "ppc": rng.choice([1, 2, 4]), "sort": -1,
                "steps": rng.randint(5, 16)}
    if kind == "window":
        return {"kind": kind, "nx": _log_int(rng, 300, 1400), "nz": _log_int(rng, 60, 300),
                "ppc": rng.choice([2, 8, 32]), "sort": -1, "steps": rng.choice([16, 24, 32])}
    if kind == "adjoint":
        plasma = rng.choice(["cold", "anisotropic"])
        nx, ny, nz = (_log_int(rng, 16, 96) for _ in range(3))
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "ppc": 16, "plasma": plasma,
                "sorted": plasma == "anisotropic", "steps": rng.randint(4, 12),
                "every": rng.choice([3, 4, 5, 10])}
    if kind == "guide":
        nx = _log_int(rng, 12, 120)
        return {"kind": kind, "nx": nx, "ny": max(6, nx // 2), "nz": _log_int(rng, 300, 3600),
                "steps": rng.randint(20, 60)}
    nx, ny, nz = (_log_int(rng, 16, 128) for _ in range(3))
    return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "ppc": rng.choice([2, 4, 8]),
            "plasma": rng.choice(["thermal", "anisotropic"]), "order": rng.choice([1, 1, 2]),
            "sort": -1, "steps": 1}


# ---------------------------------------------------------------------------
# Inputs (the same for prepare and exact): grid, sources, fields, particles
# ---------------------------------------------------------------------------
def _courant(d):
    return 0.5 / math.sqrt(sum(1.0 / x ** 2 for x in d))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (int(seed) + 1))
    return g


def _cells(n, lo=0):
    """Cell indices (x fastest) of the cells with x >= lo."""
    k, j, i = torch.meshgrid(torch.arange(n[2], device=DEV), torch.arange(n[1], device=DEV),
                             torch.arange(lo, n[0], device=DEV), indexing="ij")
    return torch.stack([i.reshape(-1), j.reshape(-1), k.reshape(-1)], 1)


def _random_in_cells(g, n, d, ppc):
    c = _cells(n).repeat_interleave(ppc, 0)
    pos = torch.rand(c.shape, generator=g, device=DEV, dtype=torch.float64)
    pos += c
    pos *= torch.tensor(d, device=DEV, dtype=torch.float64)
    for a in range(3):  # (i + frac) d may round up to the box's length
        pos[:, a].clamp_(max=float(np.nextafter(n[a] * d[a], 0.0)))
    return pos


def _lattice_points(n, per, lo=0):
    """Quiet lattice, per cell offsets (m + 1/2)/p, in cell units, cells x fastest."""
    o = [(torch.arange(p, device=DEV, dtype=torch.float64) + 0.5) / p for p in per]
    oz, oy, ox = torch.meshgrid(o[2], o[1], o[0], indexing="ij")
    local = torch.stack([ox.reshape(-1), oy.reshape(-1), oz.reshape(-1)], 1)
    return (_cells(n, lo)[:, None, :] + local[None]).reshape(-1, 3)


def _normal(g, count, sigma):
    u = torch.randn((count, 3), generator=g, device=DEV, dtype=torch.float64)
    return u.mul_(torch.tensor(sigma, device=DEV, dtype=torch.float64))


def _plasma(case, g, n, d):
    """[(q, m, w, pos, u, wpp)] and the background of the periodic plasmas."""
    ppc, kind = case["ppc"], case["plasma"]
    w = 1.0 / ppc
    if kind == "cold":
        pos = _lattice_points(n, (4, 2, ppc // 8)) * torch.tensor(d, device=DEV, dtype=torch.float64)
        u = _normal(g, pos.shape[0], (1e-4,) * 3)
        ph = float(torch.rand(1, generator=g, device=DEV)) * 2 * math.pi
        u[:, 0] += 1e-2 * torch.sin(2 * math.pi * pos[:, 0] / (n[0] * d[0]) + ph)
        return [(-1.0, 1.0, w, pos, u, None)], 1.0
    pos = _random_in_cells(g, n, d, ppc)
    N = pos.shape[0]
    if kind == "langmuir":
        u = _normal(g, N, (0.01,) * 3)
        u[:, 0] += 1e-3 * torch.sin(2 * math.pi * pos[:, 0] / (n[0] * d[0]))
        return [(-1.0, 1.0, w, pos, u, None)], 1.0
    if kind == "anisotropic":
        return [(-1.0, 1.0, w, pos, _normal(g, N, (0.25, 0.05, 0.05)), None)], 1.0
    vp = 0.05 / math.sqrt(M_PROTON)
    return [(-1.0, 1.0, w, pos, _normal(g, N, (0.05,) * 3), None),
            (1.0, M_PROTON, w, pos.clone(), _normal(g, N, (vp,) * 3), None)], 0.0


def _pulse(n, d, bc, dt, a0, w0, tau, xc, zc, yc=None):
    """E, B^{-1/2} of a pulse polarised along y travelling along +x."""
    ext = [n[a] + (bc[a] != PERIODIC) for a in range(3)]
    ax = [torch.arange(e, device=DEV, dtype=torch.float64) for e in ext]

    def at(sx, sy, t):
        x = (ax[0] + sx) * d[0] - xc - t
        y = (ax[1] + sy) * d[1]
        z = ax[2] * d[2]
        f = a0 * torch.exp(-2 * math.log(2.0) * (x / tau) ** 2) * torch.sin(x)
        r2 = ((z - zc) ** 2)[:, None] + (0.0 * y if yc is None else (y - yc) ** 2)[None, :]
        v = f[None, None, :] * torch.exp(-r2 / w0 ** 2)[:, :, None]
        for a, s in enumerate((sx, sy, 0.0)):  # padding of half-cell entries, walls
            if bc[a] == PERIODIC:
                continue
            sl = [slice(None)] * 3
            sl[2 - a] = [n[a]] if s else [0, n[a]]
            v[tuple(sl)] = 0.0
        return v

    E = torch.zeros((3, ext[2], ext[1], ext[0]), device=DEV, dtype=torch.float64)
    B = torch.zeros_like(E)
    E[1] = at(0.0, 0.5, 0.0)
    B[2] = at(0.5, 0.5, -0.5 * dt)
    return E, B


def _inputs(case, seed):
    """Everything the pass starts from, as plain values and FP64 tensors."""
    g = _gen(seed)
    kind = case["kind"]
    inp = {"laser": None, "port": None, "window": None, "filter": None, "E": None, "B": None,
           "species": [], "bg": 0.0}
    if kind == "guide":
        # TE10 guide of 3 cm x 1.5 cm x 1 m at 9 GHz, nodes per axis as given
        n = (case["nx"] - 1, case["ny"] - 1, case["nz"] - 1)
        d = (3.0 / n[0], 1.5 / n[1], 100.0 / n[2])
        bc, dt = (PEC, PEC, ABSORBING), _courant(d)
        omega = 2 * math.pi * 9.0 / 29.9792458
        inp["port"] = {"axis": 2, "plane": 0, "comp": 1, "prof": 0, "e0": 1.0, "omega": omega,
                       "tau": 2.0 * 2 * math.pi / omega}
        # a guided wave with a random envelope already inside
        beta = math.sqrt(max(omega ** 2 - (math.pi / 3.0) ** 2, 0.1))
        amp, ph = (float(v) for v in torch.rand(2, generator=g, device=DEV))
        ext = [m + 1 for m in n]
        x = torch.arange(ext[0], device=DEV, dtype=torch.float64) * d[0]
        z = torch.arange(ext[2], device=DEV, dtype=torch.float64) * d[2]
        E = torch.zeros((3, ext[2], ext[1], ext[0]), device=DEV, dtype=torch.float64)
        prof = torch.sin(math.pi * torch.minimum(x, 3.0 - x) / 3.0).clamp_(min=0.0)
        env = (0.5 + amp) * torch.sin(beta * z + 2 * math.pi * ph) * torch.exp(-((z - 50) / 30) ** 2)
        E[1] = (env[:, None] * prof[None, :])[:, None, :]
        E[1, :, n[1], :] = 0.0
        inp["E"], inp["B"] = E, torch.zeros_like(E)
    elif kind == "box":
        n, d, bc = (case["nx"], case["ny"], case["nz"]), (0.05, 0.2, 0.2), (ABSORBING,) * 3
        dt, ppc = _courant(d), case["ppc"]
        lo, ramp = n[0] // 8, 40
        pos = _lattice_points(n, (ppc, 1, 1), lo)
        pos[:, 1:] += 0.25 * (torch.rand((pos.shape[0], 2), generator=g, device=DEV,
                                         dtype=torch.float64) - 0.5)
        wpp = 0.01 * ((pos[:, 0] - lo) / ramp).clamp(0.0, 1.0) * (d[0] * d[1] * d[2] / ppc)
        pos *= torch.tensor(d, device=DEV, dtype=torch.float64)
        u = _normal(g, pos.shape[0], (1e-3,) * 3)
        L = [n[a] * d[a] for a in range(3)]
        sh = [float(v) for v in torch.rand(3, generator=g, device=DEV)]
        inp["laser"] = {"a0": 2.0, "w0": 8.0, "tau": 10.0, "t0": 0.3 + sh[0], "omega0": 1.0,
                        "yc": 0.5 * L[1], "zc": 0.5 * L[2], "i_s": 1, "slab": False}
        inp["E"], inp["B"] = _pulse(n, d, bc, dt, 2.0, 8.0, 10.0, (0.4 + 0.2 * sh[1]) * L[0],
                                    0.5 * L[2] + sh[2] - 0.5, 0.5 * L[1])
        inp["species"] = [(-1.0, 1.0, 0.01 * d[0] * d[1] * d[2] / ppc, pos, u, wpp)]
    elif kind == "window":
        # laser units of an 0.8 um pulse in a 3e18 cm^-3 plasma; the box is
        # 3 x 1 x 3 plasma wavelengths over 1400 x 2 x 300 cells
        per = {2: (1, 2, 1), 8: (2, 2, 2), 32: (4, 2, 4)}[case["ppc"]]
        c, e, me, eps0 = 299792458.0, 1.602176634e-19, 9.1093837015e-31, 8.8541878128e-12
        om0 = 2 * math.pi * c / 0.8e-6
        npl = 3.0e18 / (eps0 * me * om0 ** 2 / e ** 2 * 1e-6)
        lp = 2 * math.pi / math.sqrt(npl)
        d = (3.0 * lp / 1400.0, 1.0 * lp / 2.0, 3.0 * lp / 300.0)
        n, bc = (case["nx"], 2, case["nz"]), (ABSORBING, PERIODIC, ABSORBING)
        dt = _courant(d)
        w = npl * d[0] * d[1] * d[2] / case["ppc"]
        pos = _lattice_points(n, per) * torch.tensor(d, device=DEV, dtype=torch.float64)
        u = _normal(g, pos.shape[0], (1e-3,) * 3)
        L = [n[a] * d[a] for a in range(3)]
        sh = [float(v) for v in torch.rand(3, generator=g, device=DEV)]
        tau = 28e-15 * om0
        inp["laser"] = {"a0": 3.0, "w0": 12e-6 * om0 / c, "tau": tau, "t0": sh[0], "omega0": 1.0,
                        "yc": 0.5 * L[1], "zc": 0.5 * L[2], "i_s": 1, "slab": True}
        inp["window"] = {"axis": 0, "cells": 8, "velocity": 1.0, "t_start": 0.0, "per": per, "w": w}
        inp["E"], inp["B"] = _pulse(n, d, bc, dt, 3.0, 12e-6 * om0 / c, tau,
                                    (0.5 + 0.1 * sh[1]) * L[0], 0.5 * L[2] + sh[2] - 0.5)
        inp["species"] = [(-1.0, 1.0, w, pos, u, None)]
        inp["bg"] = npl
    else:
        n, d, bc = (case["nx"], case["ny"], case["nz"]), (1.0, 1.0, 1.0), (PERIODIC,) * 3
        dt = _courant(d)
        inp["species"], inp["bg"] = _plasma(case, g, n, d)
        if case.get("passes") or case.get("comp"):
            inp["filter"] = (case["passes"], case["comp"])
    inp.update(n=n, d=d, bc=bc, dt=dt)
    return inp


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def _make_sim(case, inp, precision="fp32", sort=-1, order=1):
    """A Sim of the case's set-up.  The particles are on the GPU already, so the
    species are declared with one particle and the capacity of all of them, and
    loaded through the C ABI from device memory."""
    from paper_2609_16575_amd import workloads as W
    from paper_2609_16575_amd.sim import Sim
    species, count = [], 0
    for q, m, w, pos, _u, wpp in inp["species"]:
        count = max(count, pos.shape[0])
        species.append(W.SpeciesInit("s", q, m, w, np.zeros((1, 3)), np.zeros((1, 3)),
                                     None if wpp is None else np.zeros(1)))
    wl = W.Workload(case["kind"], tuple(inp["n"]), tuple(inp["d"]), inp["dt"], tuple(inp["bc"]),
                    species, rho_bg=inp["bg"])
    L, P, V = inp["laser"], inp["port"], inp["window"]
    if L:
        wl.laser = W.LaserInit(L["a0"], L["w0"], L["tau"], L["t0"], L["omega0"], L["yc"], L["zc"],
                               L["i_s"], L["slab"])
    if P:
        wl.port = W.PortInit(P["axis"], P["plane"], P["comp"], P["prof"], P["e0"], P["omega"],
                             P["tau"])
    if V:
        wl.window = W.WindowInit(V["axis"], V["cells"], V["velocity"], V["t_start"],
                                 [(0, V["per"], V["w"])])
    wl.filter = inp["filter"]
    slack = 0.0 if V else float(max(count - 1, 0))
    sim = Sim(wl, precision=precision, sort_every=sort, capacity_slack=slack, shape_order=order)
    for i, (_q, _m, _w, pos, u, wpp) in enumerate(inp["species"]):
        _check(sim, sim.L.empic_load_particles_f64(
            sim.h, i, pos.shape[0], pos.data_ptr(), u.data_ptr(),
            None if wpp is None else wpp.data_ptr(), None))
    if inp["E"] is not None:
        sim.E.copy_(inp["E"])
        sim.B.copy_(inp["B"])
    return sim


def _check(sim, status):
    if status:
        raise RuntimeError(sim.L.empic_last_error(sim.h))


class _Dump:
    """Reads a species into the program's own arrays, ordered by id: momenta,
    and displacements from the start wrapped to the box."""

    def __init__(self, sim, sp, pos0, inp, spare=0):
        cap, N = sim.caps[sp], pos0.shape[0]
        self.sim, self.sp, self.rows = sim, sp, N + spare
        self.pos = torch.empty((cap, 3), dtype=torch.float64, device=DEV)
        self.u = torch.empty((cap, 3), dtype=torch.float64, device=DEV)
        self.ids = torch.empty(cap, dtype=torch.int32, device=DEV)
        self.ref, self.len = _reference(pos0, inp, self.rows)
        self.walled = any(b != PERIODIC for b in inp["bc"])

    def __call__(self):
        sim, cnt = self.sim, C.c_int64()
        _check(sim, sim.L.empic_store_particles_f64(
            sim.h, self.sp, self.pos.data_ptr(), self.u.data_ptr(), self.ids.data_ptr(),
            C.byref(cnt)))
        n = cnt.value
        ids = self.ids[:n].long()
        rows = self.rows
        if self.walled:  # removed particles and late injections: a row of their own
            ids = torch.where((ids >= 0) & (ids < rows), ids, rows)
            x = torch.zeros((rows + 1, 3), dtype=torch.float32, device=DEV)
            u = torch.zeros((rows + 1, 3), dtype=torch.float32, device=DEV)
            x[ids] = self.pos[:n].float()
            u[ids] = self.u[:n].float()
            x, u = x[:rows], u[:rows]
        else:
            x = torch.empty((rows, 3), dtype=torch.float32, device=DEV)
            u = torch.empty((rows, 3), dtype=torch.float32, device=DEV)
            x[ids] = self.pos[:n].float()
            u[ids] = self.u[:n].float()
        return x.sub_(self.ref).remainder_(self.len), u


def _reference(pos0, inp, rows):
    """(x0 - L/2 per particle, L): remainder(x - x0 + L/2, L) is the displacement
    plus half a box; walled axes (and removed particles) take a length that
    never wraps."""
    L = torch.tensor([n * d * (1.0 if b == PERIODIC else 4.0)
                      for n, d, b in zip(inp["n"], inp["d"], inp["bc"])],
                     device=DEV, dtype=torch.float64)
    ref = torch.zeros((rows, 3), device=DEV, dtype=torch.float64)
    ref[:pos0.shape[0]] = pos0
    ref -= 0.5 * L
    return ref.float(), L.float()


def _spare_rows(case, inp):
    """Rows for the particles injected during the first passes."""
    V = inp["window"]
    return V["cells"] * 2 * case["nz"] * case["ppc"] * 8 if V else 0


def prepare(case, seed):
    inp = _inputs(case, seed)
    kind = case["kind"]
    st = {"kind": kind, "steps": case["steps"]}
    if kind == "tick":
        sim = _make_sim(case, inp, case["precision"], case["sort"])
        st["fp64"] = case["precision"] == "fp64"
    elif kind in ("steps", "box"):
        sim = _make_sim(case, inp, "fp32", case["sort"], case.get("order", 1))
        sim.sort()
        st["saved"] = sim.save_state()
        st["dump"] = [_Dump(sim, i, s[3], inp) for i, s in enumerate(inp["species"])]
    elif kind == "window":
        sim = _make_sim(case, inp, "fp32", case["sort"])
        st["dump"] = [_Dump(sim, 0, inp["species"][0][3], inp, _spare_rows(case, inp))]
    elif kind == "adjoint":
        sim = _make_sim(case, inp, "fp32", 0)
        sim.sort()
        st["saved"] = sim.save_state()
        st["E0"], st["B0"] = torch.zeros_like(sim.E), torch.zeros_like(sim.B)
        st["U0"] = sim.current_buffers(0)["u"].clone()
        st["ids"] = st["saved"]["id"][0][:inp["species"][0][3].shape[0]].long()
        st["every"], st["sorted"] = case["every"], case["sorted"]
        st["dV"] = inp["d"][0] * inp["d"][1] * inp["d"][2]
    elif kind == "guide":
        sim = _make_sim(case, inp, "fp32", 0)
    else:
        sim = _make_sim(case, inp, "fp32", case["sort"], case["order"])
        sim.sort()
        sim.diagnostics()
    st["sim"] = sim
    st["counts"] = [s[3].shape[0] for s in inp["species"]]
    torch.cuda.synchronize()
    return st


def run(st):
    sim, kind = st["sim"], st["kind"]
    if kind == "tick":
        sim.step(st["steps"])
        out = {"E": sim.E, "B": sim.B, "J": sim.J}
        for i in range(len(st["counts"])):
            b = sim.current_buffers(i)
            if st["fp64"]:  # the plain path keeps its particles in order
                out["x%d" % i], out["u%d" % i] = b["pos"], b["u"]
                continue
            n = st["counts"][i]
            ids = b["id"][:n].long()
            for k in ("cell", "pos", "u"):
                o = torch.empty_like(b[k][..., :n])
                o[..., ids] = b[k][..., :n]
                out["%s%d" % (k, i)] = o
        return out
    if kind in ("steps", "box", "window"):
        if "saved" in st:
            sim.load_state(st["saved"])
        sim.step(st["steps"])
        out = {"E": sim.E, "B": sim.B, "J": sim.J}
        for i, d in enumerate(st["dump"]):
            out["x%d" % i], out["u%d" % i] = d()
        return out
    if kind == "adjoint":
        from paper_2609_16575_amd import autograd
        sim.load_state(st["saved"])
        E0 = st["E0"].detach().requires_grad_(True)
        B0 = st["B0"].detach().requires_grad_(True)
        U0 = st["U0"].detach().requires_grad_(True)
        E, B = autograd.run(sim, st["steps"], st["every"], E0, B0, [U0], sort=st["sorted"])
        loss = 0.5 * st["dV"] * ((E * E).sum() + (B * B).sum())
        gE, gB, gU = torch.autograd.grad(loss, [E0, B0, U0])
        gu = torch.empty((3, st["ids"].shape[0]), dtype=gU.dtype, device=DEV)
        gu[:, st["ids"]] = gU[:, :st["ids"].shape[0]]
        return {"E": E.detach(), "B": B.detach(), "gE": gE, "gB": gB, "gU": gu}
    sim.step(st["steps"])
    if kind == "guide":
        return {"E": sim.E, "B": sim.B}
    dg = sim.diagnostics()
    keys = ("U_E", "U_B", "U_tot", "K", "K_minus", "K_plus", "n_particles")
    return {"E": sim.E, "B": sim.B, "J": sim.J, "diag": {k: dg[k] for k in keys}}


def work(case):
    """Bytes and operations of a pass: per step every particle's and field's
    state read and written once (FP32: 28 + 28 B per particle, weights read; E,
    B read and written, J written), plus loading the saved state and the dump
    where the pass has them; order-1 push about 250 operations per particle."""
    kind, K = case["kind"], case["steps"]
    cells = case["nx"] * case.get("ny", 2) * case["nz"]
    if kind == "guide":
        return {"bytes": 48.0 * cells * K, "flops": 36.0 * cells * K}
    N = cells * case["ppc"] * (2 if case.get("plasma") == "thermal" else 1)
    if kind == "box":
        N = (case["nx"] - case["nx"] // 8) * case["ny"] * case["nz"] * case["ppc"]
    es = 2.0 if case.get("precision") == "fp64" else 1.0
    part = (60.0 if kind == "box" else 56.0) if es == 1.0 else 96.0
    fl = 250.0 if case.get("order", 1) == 1 else 900.0
    b, f = K * (part * N + 60.0 * es * cells), K * (fl * N + 40.0 * cells)
    if kind in ("steps", "box", "window"):
        b += (32.0 + 24.0) * N + 36.0 * cells  # the dump
        if kind != "window":
            b += 2 * ((36.0 if kind == "box" else 32.0) * N + 24.0 * cells)
    if kind == "adjoint":
        # forward; the states between checkpoints once more; per reversed step
        # the state and both particle adjoints read and the adjoints written
        b += b + K * ((28.0 + 24.0 + 24.0) * N + 72.0 * cells) + 2 * 32.0 * N
        f += f + K * 600.0 * N
    if kind == "monitor":
        b += 2 * 28.0 * N + (24.0 + 12.0 + 24.0 + 16.0) * cells  # particles for rho, for K+; grids
        f += 200.0 * N
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The same passes in plain torch FP64
# ---------------------------------------------------------------------------
class _Plain:
    """The PIC cycle on global FP64 positions (cell units), unsorted."""

    def __init__(self, inp, order=1):
        self.n, self.d, self.bc, self.dt = inp["n"], inp["d"], inp["bc"], inp["dt"]
        self.ext = [self.n[a] + (self.bc[a] != PERIODIC) for a in range(3)]
        self.st = [1, self.ext[0], self.ext[0] * self.ext[1]]
        self.order, self.inp, self.nstep, self.shifts = order, inp, 0, 0
        shape = (3, self.ext[2], self.ext[1], self.ext[0])
        f64 = dict(device=DEV, dtype=torch.float64)
        self.E = torch.zeros(shape, **f64) if inp["E"] is None else inp["E"].clone()
        self.B = torch.zeros(shape, **f64) if inp["B"] is None else inp["B"].clone()
        self.J = torch.zeros(shape, **f64)
        self.scale = torch.tensor(self.d, **f64)
        self.sp = []
        for q, m, w, pos, u, wpp in inp["species"]:
            alive = torch.ones(pos.shape[0], dtype=torch.bool, device=DEV)
            self.sp.append({"q": q, "m": m, "w": w if wpp is None else wpp, "x": pos / self.scale,
                            "u": u.clone(), "alive": alive})
        self.maskB = [self._mask(lambda a, c: a != c, c) for c in range(3)]
        self.maskE = [self._mask(lambda a, c: a == c, c, True) for c in range(3)]

    def _mask(self, half, c, walls=False):
        m = torch.ones(tuple(reversed(self.ext)), dtype=torch.bool, device=DEV)
        for a in range(3):
            if self.bc[a] == PERIODIC:
                continue
            sl = [slice(None)] * 3
            if half(a, c):
                sl[2 - a] = self.n[a]
                m[tuple(sl)] = False
            elif walls and a != c:
                sl[2 - a] = [0, self.n[a]]
                m[tuple(sl)] = False
        return m

    def curl(self, F, up):
        def diff(f, a):
            g = torch.roll(f, -1 if up else 1, 2 - a)
            return (g - f if up else f - g) / self.d[a]
        return torch.stack([diff(F[2], 1) - diff(F[1], 2), diff(F[0], 2) - diff(F[2], 0),
                            diff(F[1], 0) - diff(F[0], 1)])

    def faraday(self):
        """(B^{n+1/2}, centred B)."""
        new = self.B - self.dt * self.curl(self.E, True)
        new = torch.stack([torch.where(self.maskB[c], new[c], self.B[c]) for c in range(3)])
        bar = 0.5 * (self.B + new)
        return new, torch.stack([bar[c] * self.maskB[c] for c in range(3)])

    def _index(self, i, a):
        """(linear offset, inside) of index i along axis a."""
        if self.bc[a] == PERIODIC:
            return torch.remainder(i, self.n[a]) * self.st[a], None
        ok = (i >= 0) & (i < self.ext[a])
        return i.clamp(0, self.ext[a] - 1) * self.st[a], ok

    def stencil(self, x, a, half):
        """[(offset, weight)] of one axis' interpolation points."""
        if self.order == 1:
            t = x - 0.5 if half else x
            i = torch.floor(t.detach())
            f = t - i
            pts = [(i, 1.0 - f), (i + 1, f)]
        else:
            m = torch.floor(x.detach()) if half else torch.floor(x.detach() + 0.5)
            dd = x - m - (0.5 if half else 0.0)
            pts = [(m - 1, 0.5 * (0.5 - dd) ** 2), (m, 0.75 - dd ** 2),
                   (m + 1, 0.5 * (0.5 + dd) ** 2)]
        out = []
        for i, w in pts:
            off, ok = self._index(i.long(), a)
            out.append((off, w if ok is None else w * ok))
        return out

    def gather(self, Bbar, x):
        S = [[self.stencil(x[:, a], a, h) for a in range(3)] for h in (False, True)]
        out = []
        for q in range(6):
            F = (self.E[q] if q < 3 else Bbar[q - 3]).reshape(-1)
            half = [(a == q) if q < 3 else (a != q - 3) for a in range(3)]
            px, py, pz = (S[int(half[a])][a] for a in range(3))
            s = 0.0
            for oz, wz in pz:
                for oy, wy in py:
                    oyz, wyz = oy + oz, wy * wz
                    for ox, wx in px:
                        s = s + wx * wyz * F.index_select(0, ox + oyz)
            out.append(s)
        return out[:3], out[3:]

    @staticmethod
    def cross(a, b):
        return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]

    def boris(self, s, Ep, Bp):
        r = s["q"] * self.dt / (2.0 * s["m"])
        um = [s["u"][:, a] + r * Ep[a] for a in range(3)]
        g = torch.sqrt(1.0 + um[0] ** 2 + um[1] ** 2 + um[2] ** 2)
        t = [r * Bp[a] / g for a in range(3)]
        f = 2.0 / (1.0 + t[0] ** 2 + t[1] ** 2 + t[2] ** 2)
        v = self.cross(um, t)
        up = [um[a] + v[a] for a in range(3)]
        v = self.cross(up, t)
        u = torch.stack([um[a] + f * v[a] + r * Ep[a] for a in range(3)], 1)
        return u, torch.sqrt(1.0 + (u * u).sum(1))

    def _edge(self, cell, sh, c):
        """(linear offset, inside) of the edge of component c at cell + sh."""
        off, ok = 0, None
        for a in range(3):
            i = cell[a] + sh[a]
            o, inside = self._index(i, a)
            off = off + o
            if inside is not None:
                if a == c:  # half-cell component: entry n is padding
                    inside = inside & (i < self.n[a])
                ok = inside if ok is None else ok & inside
        return off, ok

    def _add(self, c, off, ok, v):
        if ok is not None:
            v = v * ok
        if v.requires_grad:
            self.Jg[c] = self.Jg[c].index_add(0, off, v)
        else:
            self.Jg[c].index_add_(0, off, v)

    def zigzag(self, s, x1, x2):
        dV = self.d[0] * self.d[1] * self.d[2]
        amp = s["q"] * s["w"] / (self.dt * dV)
        amp = amp * s["alive"]
        i1, i2 = torch.floor(x1.detach()), torch.floor(x2.detach())
        lo, hi = torch.minimum(i1, i2) + 1, torch.maximum(i1, i2)
        xr = torch.minimum(lo, torch.maximum(hi, 0.5 * (x1 + x2)))
        for cell, a0, a1 in ((i1, x1, xr), (i2, xr, x2)):
            D = a1 - a0
            Wm = 0.5 * (a0 + a1) - cell
            ci = [cell[:, a].long() for a in range(3)]
            for c in range(3):
                b1, b2 = (c + 1) % 3, (c + 2) % 3
                base = amp * D[:, c] * self.d[c]
                cr = D[:, b1] * D[:, b2] / 12.0
                for o1 in (0, 1):
                    for o2 in (0, 1):
                        sh = [0, 0, 0]
                        sh[b1], sh[b2] = o1, o2
                        off, ok = self._edge(ci, sh, c)
                        w1 = Wm[:, b1] if o1 else 1.0 - Wm[:, b1]
                        w2 = Wm[:, b2] if o2 else 1.0 - Wm[:, b2]
                        self._add(c, off, ok, base * (w1 * w2 + (cr if o1 == o2 else -cr)))

    def ez2(self, s, x1, x2):
        """Esirkepov's current with quadratic weights on the two parts of the
        move, split where it leaves the cell of its nearest nodes."""
        dV = self.d[0] * self.d[1] * self.d[2]
        amp = s["q"] * s["w"] / (self.dt * dV)
        m1, m2 = torch.floor(x1 + 0.5), torch.floor(x2 + 0.5)
        xr = torch.where(m1 != m2, torch.maximum(m1, m2) - 0.5, 0.5 * (x1 + x2))
        one = (m1 == m2).all(1, keepdim=True)
        xr = torch.where(one, x2, xr)  # a move inside one cell is one part
        for m, a0, a1 in ((m1, x1, xr), (m2, xr, x2)):
            S0, dS = [], []
            for a in range(3):
                d0, d1 = a0[:, a] - m[:, a], a1[:, a] - m[:, a]
                w0 = [0.5 * (0.5 - d0) ** 2, 0.75 - d0 ** 2, 0.5 * (0.5 + d0) ** 2]
                w1 = [0.5 * (0.5 - d1) ** 2, 0.75 - d1 ** 2, 0.5 * (0.5 + d1) ** 2]
                S0.append(w0)
                dS.append([w1[i] - w0[i] for i in range(3)])
            idx = [[torch.remainder(m[:, a].long() - 1 + i, self.n[a]) * self.st[a]
                    for i in range(3)] for a in range(3)]
            for c in range(3):
                b, e = (c + 1) % 3, (c + 2) % 3
                run1 = -amp * self.d[c] * dS[c][0]
                run2 = run1 - amp * self.d[c] * dS[c][1]
                for ib in range(3):
                    for ie in range(3):
                        T = (S0[b][ib] * S0[e][ie] + 0.5 * dS[b][ib] * S0[e][ie] +
                             0.5 * S0[b][ib] * dS[e][ie] + dS[b][ib] * dS[e][ie] / 3.0)
                        o = idx[b][ib] + idx[e][ie]
                        self.Jg[c].index_add_(0, o + idx[c][0], run1 * T)
                        self.Jg[c].index_add_(0, o + idx[c][1], run2 * T)

    def push(self, s, Bbar):
        Ep, Bp = self.gather(Bbar, s["x"])
        u, g = self.boris(s, Ep, Bp)
        x2 = s["x"] + self.dt * u / (g[:, None] * self.scale)
        (self.zigzag if self.order == 1 else self.ez2)(s, s["x"], x2)
        cols, alive = [], s["alive"]
        for a in range(3):
            if self.bc[a] == PERIODIC:
                cols.append(x2[:, a] - self.n[a] * torch.floor(x2[:, a].detach() / self.n[a]))
            else:
                cols.append(x2[:, a])
                alive = alive & (x2[:, a] >= 0) & (x2[:, a] < self.n[a])
        s["x"], s["u"], s["alive"] = torch.stack(cols, 1), u, alive

    def smooth(self, J, passes, comp):
        for a in range(3):
            for k in range(passes + comp):
                w, c = (0.25, 0.5) if k < passes else (-0.25, 1.5)
                J = w * torch.roll(J, 1, 3 - a) + c * J + w * torch.roll(J, -1, 3 - a)
        return J

    def shift_window(self, V):
        t = self.nstep * self.dt
        a, k = V["axis"], V["cells"]
        if (t - V["t_start"]) * V["velocity"] < (self.shifts + 1) * k * self.d[a]:
            return
        self.shifts += 1
        for F, isB in ((self.E, False), (self.B, True)):
            for c in range(3):
                half = (a != c) if isB else (a == c)
                L = self.n[a] if half else self.ext[a]
                f = F[c].movedim(2 - a, 0)
                moved = f[k:L].clone()
                f.zero_()
                f[:L - k] = moved
        for s in self.sp:
            s["x"][:, a] -= k
            s["alive"] &= s["x"][:, a] >= 0
            # the new cells' lattice, x fastest over all lattice points
            n = list(self.n)
            per = V["per"]
            ax = [(torch.arange(k * per[0] if b == a else n[b] * per[b], device=DEV,
                                dtype=torch.float64) + 0.5) / per[b] for b in range(3)]
            ax[a] = ax[a] + (n[a] - k)
            z, y, x = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
            new = torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)], 1)
            s["x"] = torch.cat([s["x"], new])
            s["u"] = torch.cat([s["u"], torch.zeros_like(new)])
            s["alive"] = torch.cat([s["alive"], torch.ones(len(new), dtype=torch.bool, device=DEV)])

    def step(self):
        inp = self.inp
        if inp["window"]:
            self.shift_window(inp["window"])
        B, Bbar = self.faraday()
        self.Jg = [torch.zeros(self.E[0].numel(), device=DEV, dtype=torch.float64)
                   for _ in range(3)]
        for s in self.sp:
            self.push(s, Bbar)
        J = torch.stack(self.Jg).reshape(self.E.shape)
        if inp["filter"]:
            J = self.smooth(J, *inp["filter"])
        old, self.B, self.J = self.E, B, J
        new = old + self.dt * (self.curl(B, False) - J)
        self.E = torch.stack([torch.where(self.maskE[c], new[c], old[c]) for c in range(3)])
        if any(b != PERIODIC for b in self.bc):
            self.faces(old)
        self.nstep += 1

    def faces(self, old):
        E, inp, dt = self.E, self.inp, self.dt
        if inp["laser"]:
            L = inp["laser"]
            y = (torch.arange(self.n[1], device=DEV, dtype=torch.float64) + 0.5) * self.d[1]
            k0, k1 = (1, self.n[2]) if self.bc[2] != PERIODIC else (0, self.n[2])
            z = torch.arange(k0, k1, device=DEV, dtype=torch.float64) * self.d[2]
            r2 = ((z - L["zc"]) ** 2)[:, None] + (0.0 * y if L["slab"] else (y - L["yc"]) ** 2)[None]
            t = (self.nstep + 0.5) * dt - L["t0"]
            inc = L["a0"] * torch.exp(-r2 / L["w0"] ** 2) * (
                math.exp(-2 * math.log(2.0) * t * t / L["tau"] ** 2) * math.sin(L["omega0"] * t))
            E[1, k0:k1, :self.n[1], L["i_s"]] += dt * 2.0 * inc / self.d[0]
        for a in range(3):
            if self.bc[a] != ABSORBING:
                continue
            co = (dt - self.d[a]) / (dt + self.d[a])
            for c in range(3):
                if c == a:
                    continue
                e, o, n = E[c].movedim(2 - a, 0), old[c].movedim(2 - a, 0), self.n[a]
                e[0] = o[1] + co * (e[1] - o[0])
                e[n] = o[n - 1] + co * (e[n - 1] - o[n])
        for a in range(3):
            if self.bc[a] == PEC:
                for c in range(3):
                    if c != a:
                        e = E[c].movedim(2 - a, 0)
                        e[0] = 0.0
                        e[self.n[a]] = 0.0
        P = inp["port"]
        if P:  # along z, E_y with a half-sine profile along x
            t = (self.nstep + 1) * dt
            amp = P["e0"] * (1 - math.exp(-t / P["tau"])) * math.sin(P["omega"] * t)
            x = torch.arange(self.ext[0], device=DEV, dtype=torch.float64) * self.d[0]
            L = self.n[0] * self.d[0]
            E[1, P["plane"], :self.n[1], :] = amp * torch.sin(math.pi * torch.minimum(x, L - x) / L)

    def kinetic(self, s, u):
        uu = (u * u).sum(1)
        return float((s["w"] * s["m"] * uu / (torch.sqrt(1.0 + uu) + 1.0)).sum())

    def diagnostics(self):
        dV = self.d[0] * self.d[1] * self.d[2]
        new, Bbar = self.faraday()
        UE, UB = 0.5 * dV * float((self.E ** 2).sum()), 0.5 * dV * float((self.B * new).sum())
        km, kp = [], []
        for s in self.sp:
            km.append(self.kinetic(s, s["u"]))
            kp.append(self.kinetic(s, self.boris(s, *self.gather(Bbar, s["x"]))[0]))
        K = [0.5 * (a + b) for a, b in zip(km, kp)]
        return {"U_E": UE, "U_B": UB, "U_tot": UE + UB + sum(K), "K": K, "K_minus": km,
                "K_plus": kp, "n_particles": [int(s["alive"].sum()) for s in self.sp]}


def exact(case, seed):
    kind = case["kind"]
    cells = case["nx"] * case.get("ny", 2) * case["nz"]
    N = cells * case.get("ppc", 0) * (2 if case.get("plasma") == "thermal" else 1)
    if kind == "adjoint":
        # every step's intermediates are kept for the gradients
        if N * case["steps"] > 12_000_000:
            return None
        return _exact_adjoint(case, _inputs(case, seed))
    if N * case["steps"] * (4 if case.get("order", 1) == 2 else 1) > 1_200_000_000:
        return None  # over about 20 seconds
    inp = _inputs(case, seed)
    with torch.no_grad():
        p = _Plain(inp, case.get("order", 1))
        for _ in range(case["steps"]):
            p.step()
        out = {"E": p.E, "B": p.B, "J": p.J}
        if kind == "guide":
            return {"E": p.E, "B": p.B}
        if kind == "monitor":
            return {**out, "diag": p.diagnostics()}
        for i, s in enumerate(p.sp):
            if kind == "tick":
                if case["precision"] == "fp64":
                    pad = (len(s["x"]) + 63) // 64 * 64 - len(s["x"])
                    for k, v in (("x", s["x"] * p.scale), ("u", s["u"])):
                        out["%s%d" % (k, i)] = torch.nn.functional.pad(v, (0, 0, 0, pad)).T
                else:
                    out["cell%d" % i] = out["pos%d" % i] = None  # storage of its own
                    out["u%d" % i] = s["u"].T
                continue
            rows = inp["species"][i][3].shape[0] + _spare_rows(case, inp)
            ref, L = _reference(inp["species"][i][3], inp, rows)
            x, u = (torch.zeros((rows, 3), device=DEV, dtype=torch.float64) for _ in range(2))
            k = min(rows, len(s["x"]))
            live = s["alive"][:k, None]
            x[:k] = torch.where(live, s["x"][:k] * p.scale, 0.0)
            u[:k] = torch.where(live, s["u"][:k], 0.0)
            out["x%d" % i], out["u%d" % i] = (x - ref.double()).remainder(L.double()), u
        return out


def _exact_adjoint(case, inp):
    p = _Plain(inp)
    E0 = p.E.requires_grad_(True)
    B0 = p.B.requires_grad_(True)
    U0 = p.sp[0]["u"].requires_grad_(True)
    for _ in range(case["steps"]):
        p.step()
    dV = inp["d"][0] * inp["d"][1] * inp["d"][2]
    loss = 0.5 * dV * ((p.E ** 2).sum() + (p.B ** 2).sum())
    gE, gB, gU = torch.autograd.grad(loss, [E0, B0, U0])
    return {"E": p.E.detach(), "B": p.B.detach(), "gE": gE, "gB": gB, "gU": gU.T.contiguous()}
