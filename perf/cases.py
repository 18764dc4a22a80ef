"""The work a user of this framework has it do, as cases that can be timed.

A case names a plasma by its phase-space grid, markers per cell, storage form
and the entry point that drives it:

* ``steps``    a Simulation advanced some steps (direct launches or graph
               replay), then its field, charge density and distribution read;
* ``stages``   one step by the separate stage calls;
* ``loading``  the distribution of a given marker set (no handle, no workspace);
* ``species``  electrons and mobile ions in one field;
* ``batch``    a parameter scan of uneven instances stepped together;
* ``adjoint``  the gradient of the time-integrated field energy.

Sizes and initial distributions are those of ``paper_1804_03901_amd.inputs``.
Markers are drawn on the GPU from the seed alone (``ppc`` uniform markers per
phase cell, each carrying f0 at its own position).  ``exact`` advances the
same markers by the method's definitions in plain FP64 torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1804_03901_amd import adjoint, avl, inputs

DEV = "cuda:0"

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------


def listed():
    return [
        # the smallest run anyone starts with: linear Landau damping, 16,384
        # markers, replayed as a graph, where only latency and launches count
        {"name": "landau_64x64_fp64", "kind": "steps", "plasma": "landau", "nx": 64, "nv": 64, "ppc": 4,
         "fp32": False, "kahan": False, "steps": 10, "graph": True},
        # two small kinetic species in one field (ion-acoustic waves)
        {"name": "ion_acoustic_fp64", "kind": "species", "nx": 32, "nv": 1024, "nv_ions": 128, "ppc": 4,
         "fp32": False, "steps": 10},
        # the distribution of markers at hand, from code that cannot allocate;
        # log-uniform weights
        {"name": "loading_256x256_fp64", "kind": "loading", "nx": 256, "nv": 256, "ppc": 4, "fp32": False,
         "weights": "logu"},
        # a program that drives the stages itself, at the size of the Langmuir runs
        {"name": "stages_256x256_fp32", "kind": "stages", "plasma": "langmuir", "nx": 256, "nv": 256, "ppc": 4,
         "fp32": True},
        # electron Bernstein waves: 1D-3V with a background magnetic field
        {"name": "bernstein_64x24c_fp64", "kind": "steps", "plasma": "bernstein", "nx": 64, "nv": 24, "ppc": 2,
         "fp32": False, "kahan": False, "steps": 2, "graph": False},
        # odd sizes, direct launches, compensated FP32 sums
        {"name": "bump_512x777_kahan", "kind": "steps", "plasma": "bump", "nx": 512, "nv": 777, "ppc": 5,
         "fp32": True, "kahan": True, "steps": 5, "graph": False},
        # gradient of the time-integrated field energy, a checkpoint every 20 steps
        {"name": "adjoint_1024x512_fp32", "kind": "adjoint", "nx": 1024, "nv": 512, "ppc": 8, "fp32": True,
         "steps": 60, "every": 20},
        # the paper's Landau test with trapping: kicks of several velocity
        # cells, output quantities taken every five steps
        {"name": "paper_landau_fp64", "kind": "steps", "plasma": "paper", "nx": 512, "nv": 6600, "ppc": 4,
         "fp32": False, "kahan": False, "steps": 5, "graph": False},
        # the benchmark plasma in both storage forms
        {"name": "bump_1024x1024_fp32", "kind": "steps", "plasma": "bump", "nx": 1024, "nv": 1024, "ppc": 16,
         "fp32": True, "kahan": False, "steps": 10, "graph": True},
        {"name": "bump_1024x1024_fp64", "kind": "steps", "plasma": "bump", "nx": 1024, "nv": 1024, "ppc": 16,
         "fp32": False, "kahan": False, "steps": 10, "graph": True},
        # the 64-instance parameter scan
        {"name": "scan_64_fp32", "kind": "batch", "count": 64, "ppc": 8, "fp32": True, "steps": 5},
        # two-stream instability in 1D-3V, 67M phase cells, 268M markers
        {"name": "two_stream_256x64c_fp32", "kind": "steps", "plasma": "two_stream", "nx": 256, "nv": 64, "ppc": 4,
         "fp32": True, "kahan": False, "steps": 2, "graph": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "steps3", "stages", "loading", "species", "batch", "adjoint"])
    fp32 = rng.random() < 0.5
    if kind == "loading":
        nx = 2 ** rng.randint(3, 10)
        ppc = _log_int(rng, 2, 20)
        nv = _log_int(rng, 8, max(9, min(600, 900_000 // (nx * ppc))))
        return {"kind": kind, "nx": nx, "nv": nv, "ppc": ppc, "fp32": fp32,
                "weights": rng.choice(["analytic", "logu"])}
    if kind == "species":
        return {"kind": kind, "nx": 2 ** rng.randint(4, 8), "nv": _log_int(rng, 256, 1024),
                "nv_ions": _log_int(rng, 64, 256), "ppc": rng.randint(2, 8), "fp32": fp32, "steps": rng.randint(2, 10)}
    if kind == "batch":
        return {"kind": kind, "count": _log_int(rng, 4, 48), "ppc": rng.randint(4, 10), "fp32": fp32,
                "steps": rng.randint(1, 4)}
    if kind == "adjoint":
        steps = rng.randint(10, 40)
        return {"kind": kind, "nx": 2 ** rng.randint(6, 10), "nv": _log_int(rng, 64, 512), "ppc": rng.randint(3, 8),
                "fp32": fp32, "steps": steps, "every": rng.randint(5, 20)}
    if kind == "steps3":
        plasma = rng.choice(["two_stream", "bernstein"])
        nx = 2 ** rng.randint(5, 8)
        nv = _log_int(rng, 12, 48)
        ppc = rng.randint(2, 4)
        while nx * nv ** 3 * ppc > 60_000_000:
            nv -= 3
        return {"kind": "steps", "plasma": plasma, "nx": nx, "nv": nv, "ppc": ppc,
                "fp32": fp32 and plasma == "two_stream", "kahan": False, "steps": rng.randint(1, 2),
                "graph": rng.random() < 0.5}
    plasma = rng.choice(["bump", "bump", "langmuir", "landau", "paper"])
    nx = 2 ** rng.randint(5, 12)
    ppc = _log_int(rng, 2, 20)
    nv = _log_int(rng, max(48, nx // 8), 4000)
    while nx * nv * ppc > 16_800_000:
        nv = max(48, nv * 3 // 4)
        ppc = max(2, ppc * 3 // 4)
    case = {"kind": kind, "plasma": plasma, "nx": nx, "nv": nv, "ppc": ppc, "fp32": fp32}
    if kind == "steps":
        case.update(kahan=fp32 and rng.random() < 0.25, steps=rng.randint(1, 8), graph=rng.random() < 0.5)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _workload(case, seed):
    nx, nv, ppc = case["nx"], case["nv"], case["ppc"]
    plasma = case.get("plasma", "bump")
    if plasma == "landau":
        return inputs.landau_small().replace(nx=nx, nv=(nv, 1, 1), ppc=ppc, seed=seed)
    if plasma == "paper":
        return inputs.paper_landau(ppc=ppc, seed=seed).replace(nx=nx, nv=(nv, 1, 1))
    if plasma == "langmuir":
        return inputs.langmuir_noise(nx=nx, nv=nv, ppc=ppc, seed=seed)
    if plasma == "bernstein":
        return inputs.bernstein(nx=nx, nv=nv, ppc=ppc, seed=seed)
    if plasma == "two_stream":
        return inputs.two_stream_3v(nx=nx, nv=nv, ppc=ppc, seed=seed)
    return inputs.bump_on_tail(nx=nx, nv=nv, ppc=ppc, seed=seed, weights=case.get("weights", "analytic"))


def _workloads(case, seed):
    if case["kind"] == "species":
        return list(inputs.ion_acoustic(nx=case["nx"], nv_e=case["nv"], nv_i=case["nv_ions"], ppc=case["ppc"],
                                        seed=seed))
    if case["kind"] == "batch":
        # the scan's shapes and beams are the workload's own; the markers follow the seed
        scan = inputs.batched_scan(count=case["count"], ppc=case["ppc"])
        return [w.replace(seed=seed + 1000 * b) for b, w in enumerate(scan)]
    return [_workload(case, seed)]


def _markers(w, seed):
    """ppc uniform markers per phase cell, velocity-major, and their f0 (FP64, on the GPU)."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    uniform = lambda: torch.rand(w.n_markers, dtype=torch.float64, device=DEV, generator=gen)
    cell = torch.arange(w.n_cells, device=DEV).repeat_interleave(w.ppc)
    x = torch.remainder(((cell % w.nx) + uniform()) * w.dx, w.L)
    x[x >= w.L] = 0.0
    row = cell // w.nx
    del cell
    v = torch.empty(w.vdim, w.n_markers, dtype=torch.float64, device=DEV)
    for d in range(w.vdim):
        v[d] = w.vmin[d] + ((row % w.nv[d]) + uniform()) * w.dv(d)
        row = row // w.nv[d]
    if w.weights == "logu":
        return x, v, 10.0 ** (-8.0 + 8.0 * uniform())
    f = torch.zeros_like(x)
    for p in w.populations:
        term = torch.full_like(x, p.density)
        for d in range(w.vdim):
            s = p.vth[d]
            term *= torch.exp(-((v[d] - p.drift[d]) ** 2) / (2.0 * s * s)) / (s * math.sqrt(2.0 * math.pi))
        f += term
    dens = torch.ones_like(x)
    for m, phase in zip(w.mode_numbers, inputs.mode_phases(w)):
        dens += w.mode_amplitude * torch.cos(2.0 * math.pi / w.L * m * x + float(phase))
    return x, v, f * dens


def _precision(case):
    return avl.AVL_FP32 if case["fp32"] else avl.AVL_FP64


def prepare(case, seed):
    kind, prec = case["kind"], _precision(case)
    ws = _workloads(case, seed)
    marks = [_markers(w, seed + 17 * i) for i, w in enumerate(ws)]
    state = {"case": case}
    if kind == "batch":
        b = avl.Batch(ws, marks, precision=prec, device=DEV)
        grid = torch.float32 if case["fp32"] else torch.float64
        nx, cells = sum(w.nx for w in ws), sum(w.n_cells for w in ws)
        state.update(batch=b, instances=[b.instance(i) for i in range(len(ws))], ws=ws,
                     E=torch.empty(nx, dtype=torch.float64, device=DEV),
                     rho=torch.empty(nx, dtype=torch.float64, device=DEV),
                     f=torch.empty(cells, dtype=grid, device=DEV))
        return state
    w, (x, v, f) = ws[0], marks[0]
    if kind == "loading":
        grid = torch.float32 if case["fp32"] else torch.float64
        state.update(cfg=avl.make_config(w, prec), x=x, v=v.reshape(-1), f=f,
                     f_out=torch.empty(w.nv[0], w.nx, dtype=grid, device=DEV),
                     D_out=torch.empty(w.nv[0], w.nx, dtype=grid, device=DEV))
        return state
    sims = [avl.Simulation(w, x, v.reshape(-1), f, precision=prec, device=DEV,
                           options=avl.AVL_OPT_KAHAN32 if case.get("kahan") else 0)
            for w, (x, v, f) in zip(ws, marks)]
    state.update(sim=sims[0], sims=sims)
    if kind == "species":
        state["multi"] = avl.MultiSpecies(sims)
    elif kind == "adjoint":
        state.update(x=x, v=v.reshape(-1), f=f)
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "steps":
        sim = state["sim"]
        diag = sim.step(case["steps"], graph=case["graph"])
        E, rho = sim.field()
        out = {"diag": diag, "E": E, "rho": rho, "f": sim.reconstruct()}
        if case["plasma"] == "paper":
            quantities, j, residual = sim.diagnostics(spatial=True)
            out.update(quantities=[quantities[k] for k in ("Ee", "Ekin", "Etot", "N", "S")], j=j, residual=residual)
        return out
    if kind == "stages":
        sim = state["sim"]
        sim.push()
        sim.sort()
        f, D = sim.reconstruct(want_D=True)
        rho = sim.moments()
        E, W = sim.poisson()
        return {"f": f, "D": D, "rho": rho, "E": E, "W": W}
    if kind == "loading":
        avl.avl_reconstruct_noalloc(state["cfg"], None, state["x"], state["v"], state["f"], state["f_out"],
                                    state["D_out"])
        return {"f": state["f_out"], "D": state["D_out"]}
    if kind == "species":
        diag = state["multi"].step(case["steps"])
        fields = [sim.field() for sim in state["sims"]]
        return {"diag": diag, "E": fields[0][0], "rho": [r for _, r in fields],
                "f": [sim.reconstruct() for sim in state["sims"]]}
    if kind == "batch":
        diag = state["batch"].step(case["steps"])
        i = g = 0
        for w, inst in zip(state["ws"], state["instances"]):
            avl.avl_get_field(inst.h, state["E"][i:i + w.nx], state["rho"][i:i + w.nx])
            avl.avl_reconstruct(inst.h, state["f"][g:g + w.n_cells])
            i += w.nx
            g += w.n_cells
        return {"diag": diag, "E": state["E"], "rho": state["rho"], "f": state["f"]}
    J, grad = adjoint.energy_and_gradient(state["sim"], state["x"], state["v"], state["f"], case["steps"],
                                          case["every"])
    return {"J": J, "grad": grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Per step and marker: position, velocity and weight read, position and
    velocity written; per step the grid written.  The reverse of a step reads
    the same and updates three adjoints a marker."""
    size = 4.0 if case["fp32"] else 8.0
    total = {"bytes": 0.0, "flops": 0.0}
    for w in _workloads(case, 1):
        n, cells, corners = float(w.n_markers), float(w.n_cells), 2.0 ** (1 + w.vdim)
        moved = 1 + (w.vdim if any(w.B) else 1)
        step = {"bytes": n * size * (2 + w.vdim + moved) + cells * size, "flops": n * (16 + 6 * corners)}
        if case["kind"] == "loading":
            step = {"bytes": n * 24.0 + 2.0 * cells * size, "flops": n * (6 + 6 * corners)}
        elif case["kind"] == "adjoint":
            step = {"bytes": 2 * step["bytes"] + n * 48.0, "flops": 4 * step["flops"]}
        passes = case.get("steps", 1)
        for k in total:
            total[k] += passes * step[k]
    return total


# ---------------------------------------------------------------------------
# the same in plain FP64 torch
# ---------------------------------------------------------------------------

_CHUNK = 1 << 24


def _axis(coord, lo, h):
    t = (coord - lo) / h - 0.5
    low = torch.floor(t.detach())
    return low.to(torch.int64), t - low


def _deposit(w, x, v, f):
    """f = N / D and D on the grid: cloud-in-cell sums of f and 1 over the markers."""
    N = torch.zeros(w.n_cells, dtype=torch.float64, device=x.device)
    D = torch.zeros_like(N)
    for lo in range(0, max(1, x.numel()), _CHUNK):
        part = slice(lo, lo + _CHUNK)
        fc = f[part]
        axes = [_axis(x[part], 0.0, w.dx)] + [_axis(v[d, part], w.vmin[d], w.dv(d)) for d in range(w.vdim)]
        for corner in range(2 ** (1 + w.vdim)):
            weight, index, inside, stride = 1.0, 0, None, 1
            for d, (low, frac) in enumerate(axes):
                up = (corner >> d) & 1
                weight = weight * (frac if up else 1.0 - frac)
                j = low + up
                if d == 0:
                    j = torch.remainder(j, w.nx)
                else:
                    ok = (j >= 0) & (j < w.nv[d - 1])
                    inside = ok if inside is None else inside & ok
                    j = j.clamp(0, w.nv[d - 1] - 1)
                index = index + j * stride
                stride *= w.nx if d == 0 else w.nv[d - 1]
            weight = torch.where(inside, weight, torch.zeros_like(weight))
            N = N.index_add(0, index, weight * fc) if f.requires_grad or x.requires_grad else N.index_add_(0, index, weight * fc)
            D = D.index_add(0, index, weight) if x.requires_grad else D.index_add_(0, index, weight)
    some = D > 0
    return torch.where(some, N / torch.where(some, D, torch.ones_like(D)), torch.zeros_like(N)), D


def _charge(w, f):
    vol = 1.0
    for d in range(w.vdim):
        vol *= w.dv(d)
    return w.q * vol * f.reshape(-1, w.nx).sum(0)


def _solve(w, rho):
    """E_hat = -i c_p kappa / K^2 rho_hat with kappa = sin(k dx)/dx, K = 2 sin(k dx/2)/dx; no mean, no Nyquist."""
    m = torch.arange(w.nx // 2 + 1, dtype=torch.float64, device=rho.device)
    y = 2.0 * math.pi * m / w.nx
    K2 = (2.0 * torch.sin(0.5 * y) / w.dx) ** 2
    g = w.c_p * (torch.sin(y) / w.dx) / torch.where(K2 > 0, K2, torch.ones_like(K2))
    g[0] = 0.0
    g[-1] = 0.0
    return torch.fft.irfft(torch.fft.rfft(rho - rho.mean()) * (-1j * g), n=w.nx)


def _push(w, x, v, E):
    low, a = _axis(x, 0.0, w.dx)
    i = torch.remainder(low, w.nx)
    el = (1.0 - a) * E[i] + a * E[torch.remainder(i + 1, w.nx)]
    qm = w.q / w.m
    if any(w.B):
        h, t = 0.5 * qm * el * w.dt, [0.5 * qm * w.dt * b for b in w.B]
        s = 2.0 / (1.0 + sum(c * c for c in t))
        ux, uy, uz = v[0] + h, v[1], v[2]
        px, py, pz = ux + (uy * t[2] - uz * t[1]), uy + (uz * t[0] - ux * t[2]), uz + (ux * t[1] - uy * t[0])
        v = torch.stack([ux + s * (py * t[2] - pz * t[1]) + h, uy + s * (pz * t[0] - px * t[2]),
                         uz + s * (px * t[1] - py * t[0])])
    elif w.vdim == 3:
        v[0] += qm * el * w.dt
    else:
        v = v + (qm * el * w.dt)[None]
    x = x + v[0] * w.dt
    return torch.where(x.detach() - w.L * torch.floor(x.detach() / w.L) < w.L, x - w.L * torch.floor(x.detach() / w.L),
                       torch.zeros_like(x)), v


def _mode1(w, E):
    phase = 2.0 * math.pi * torch.arange(w.nx, dtype=torch.float64, device=E.device) / w.nx
    return 2.0 / w.nx * torch.sqrt((E * torch.cos(phase)).sum() ** 2 + (E * torch.sin(phase)).sum() ** 2)


def _energy(w, E):
    return (E * E).sum() * w.dx / (2.0 * w.c_p)


def _advance(ws, marks, steps):
    """Steps of one or several species in one field: per species f and rho, the field, W and mode 1 per step."""
    grids = [_deposit(w, *m)[0] for w, m in zip(ws, marks)]
    rho = [_charge(w, g) for w, g in zip(ws, grids)]
    E = _solve(ws[0], sum(rho))
    marks, diag = list(marks), []
    for _ in range(steps):
        for s, w in enumerate(ws):
            x, v, f = marks[s]
            x, v = _push(w, x, v, E)
            marks[s] = (x, v, f)
            grids[s] = _deposit(w, x, v, f)[0]
            rho[s] = _charge(w, grids[s])
        E = _solve(ws[0], sum(rho))
        diag.append(torch.stack([_energy(ws[0], E), _mode1(ws[0], E)]))
    return marks, grids, rho, E, torch.stack(diag) if diag else None


def _shaped(w, f):
    return f.reshape(tuple(w.nv[d] for d in reversed(range(w.vdim))) + (w.nx,))


def exact(case, seed):
    kind = case["kind"]
    ws = _workloads(case, seed)
    if kind == "batch":
        parts = []
        for i, w in enumerate(ws):
            _, grids, rho, E, diag = _advance([w], [_markers(w, seed + 17 * i)], case["steps"])
            parts.append((diag, E, rho[0], grids[0]))
        diag, E, rho, f = zip(*parts)
        return {"diag": torch.stack(diag), "E": torch.cat(E), "rho": torch.cat(rho), "f": torch.cat(f)}
    marks = [_markers(w, seed + 17 * i) for i, w in enumerate(ws)]
    w = ws[0]
    if kind == "loading":
        f, D = _deposit(w, *marks[0])
        return {"f": _shaped(w, f), "D": _shaped(w, D)}
    if kind == "adjoint":
        x, v, f = marks[0]
        f.requires_grad_(True)
        E = _solve(w, _charge(w, _deposit(w, x, v, f)[0]))
        J = 0.0
        for _ in range(case["steps"]):
            x, v = _push(w, x, v, E)
            E = _solve(w, _charge(w, _deposit(w, x, v, f)[0]))
            J = J + (E * E).sum() * w.dx * w.dt
        J.backward()
        return {"J": J.detach(), "grad": f.grad}
    marks, grids, rho, E, diag = _advance(ws, marks, 1 if kind == "stages" else case["steps"])
    if kind == "species":
        return {"diag": diag, "E": E, "rho": rho, "f": [_shaped(s, g) for s, g in zip(ws, grids)]}
    f = _shaped(w, grids[0])
    if kind == "stages":
        return {"f": f, "D": _shaped(w, _deposit(w, *marks[0])[1]), "rho": rho[0], "E": E,
                "W": _energy(w, E).reshape(1)}
    out = {"diag": diag, "E": E, "rho": rho[0], "f": f}
    if case["plasma"] == "paper":
        centre = w.vmin[0] + (torch.arange(w.nv[0], dtype=torch.float64, device=DEV) + 0.5) * w.dv(0)
        cell = w.dx * w.dv(0)
        ekin = 0.5 * w.m * float((f.sum(1) * centre ** 2).sum()) * cell
        ee = float(_energy(w, E))
        entropy = float(torch.special.xlogy(f, f).sum()) * cell
        div = (torch.roll(E, -1) - torch.roll(E, 1)) / (2.0 * w.dx * w.c_p)
        out.update(quantities=[ee, ekin, ee + ekin, float(f.sum()) * cell, entropy],
                   j=w.q * w.dv(0) * (f * centre[:, None]).sum(0), residual=(rho[0] - rho[0].mean()) - div)
    return out
