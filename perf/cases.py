"""The work a simulation code gives this library, as cases that can be timed.

A step of such a code assigns the particles to the mesh, solves the
brane-bending mode on the domain grid and on its refinements, fills refinement
boundaries from their parents and differences the potentials; these cases are
those calls through the Python binding, from 32^3 cells (latency) to 512^3
(bandwidth), with both precisions, both deposit schemes, cubic and ragged
shapes, tuned and default schedules.  Arrays are float64 on the GPU, as the
binding takes them; inputs are synthetic fields with the statistics of the
benchmark workloads (top-hat, lognormal, Zel'dovich particles), made from the
seed on the GPU.
"""
from __future__ import annotations

import math
import os
import random
import shutil
import tempfile

import torch

from paper_1303_0008_amd import vmg

HERE = os.path.dirname(os.path.abspath(__file__))
TUNE_FILE = os.path.join(os.path.dirname(HERE), "paper_1303_0008_amd", "tune_gfx950.txt")
KAPPA = 1.5                    # source coefficient of every workload
ZELDOVICH_AMPLITUDE = 1.2      # displacement of the 256^3 particle workload
SCHEMES = {"cic": vmg.ASSIGN_CIC, "tsc": vmg.ASSIGN_TSC}
PRECISIONS = {"fp64": vmg.FP64, "mixed": vmg.MIXED}


def _solve(name, n, prec, field, alpha, tol, sigma=1.0, tuned=True, kept=True):
    c = {"kind": "solve", "n0": n[0], "n1": n[1], "n2": n[2], "prec": prec, "field": field, "alpha": alpha,
         "tol": tol, "sigma": sigma, "tuned": tuned, "kept": kept}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest calls: a small domain solved again and again on a plan the
        # program keeps (spherical test problem of Sec. IV.C) ...
        _solve("solve32_fp64", (32, 32, 32), "fp64", "tophat", 0.05, 1e-10),
        # ... and the one-call convenience with default schedules, whose plan
        # lives for one solve
        _solve("field64_fp64", (64, 64, 64), "fp64", "lognormal", 0.1, 1e-8, tuned=False, kept=False),
        # ordinary domain grids of a time-stepping program, graph replay and the
        # committed schedules; both precisions
        _solve("solve128_mixed", (128, 128, 128), "mixed", "lognormal", 0.1, 1e-8),
        _solve("solve256_fp64", (256, 256, 256), "fp64", "zeldovich", 0.2, 1e-8),
        # the largest domain grid of the benchmark
        _solve("solve512_mixed", (512, 512, 512), "mixed", "lognormal", 0.2, 1e-8, sigma=1.5),
        # one batch of refinement patches of uneven sizes, and the interpolation
        # of their ghost shells and initial guesses from the parent
        {"name": "patches96_mixed", "kind": "patches", "count": 96, "sides": "24,16,32,48,64", "ragged": False,
         "parent": 128, "ratio": 4, "prec": "mixed", "alpha": 0.1, "sigma": 1.5, "tol": 1e-8, "tuned": True},
        {"name": "fills96", "kind": "fills", "count": 96, "sides": "24,16,32,48,64", "ragged": False, "parent": 256,
         "ratio": 2},
        # a domain grid with two depths of refinements, solved top down
        {"name": "levels128_mixed", "kind": "levels", "n": 128, "refinements": 8, "side": 64, "prec": "mixed",
         "alpha": 0.2, "tol": 1e-8, "tuned": True},
        # particles to mesh: the benchmark's 256^3 lattice-ordered particles, a
        # small cloud-in-cell deposit of unordered particles, a refinement's mesh
        {"name": "assign256_tsc", "kind": "assign", "lattice": 256, "n0": 256, "n1": 256, "n2": 256,
         "scheme": "tsc", "shuffled": False},
        {"name": "assign64_cic", "kind": "assign", "lattice": 64, "n0": 64, "n1": 64, "n2": 64, "scheme": "cic",
         "shuffled": True},
        {"name": "region64_tsc", "kind": "region", "lattice": 192, "n0": 64, "n1": 64, "n2": 64, "box": 384,
         "scheme": "tsc", "shuffled": False},
        # potentials to forces on the benchmark grid
        {"name": "force256", "kind": "force", "n0": 256, "n1": 256, "n2": 256},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: default schedules (what a size without tuning gets), ragged
    shapes; domain grids of 32^3 to about 320^3 cells (any c 2^k with c = 4..8 per
    axis coarsens), 8 to 128 patches, 2e4 to 1.6e7 particles on meshes of 24 to
    256 cells per axis."""
    kind = rng.choice(["solve", "solve", "solve", "solve", "patches", "patches", "fills", "levels", "assign",
                       "assign", "assign", "region", "force"])
    if kind == "solve":
        while True:
            s = 1 << rng.choice([3, 3, 4, 4, 5, 5, 6])
            n = tuple(rng.randint(4, 8) * s for _ in range(3))
            if n[0] * n[1] * n[2] <= 1 << 25:
                break
        prec = rng.choice(["fp64", "mixed"])
        return _solve(None, n, prec, "lognormal", rng.choice([0.05, 0.1, 0.2]),
                      rng.choice([1e-8, 1e-8, 1e-9] if prec == "mixed" else [1e-8, 1e-9, 1e-10]),
                      sigma=round(rng.uniform(0.6, 1.4), 2), tuned=False, kept=rng.random() < 0.75)
    if kind == "patches":
        return {"kind": "patches", "count": _log_uniform(rng, 8, 128), "ragged": True,
                "parent": rng.choice([64, 96, 128]), "ratio": rng.choice([2, 4]),
                "prec": rng.choice(["fp64", "mixed"]), "alpha": rng.choice([0.05, 0.1]),
                "sigma": round(rng.uniform(0.8, 1.5), 2), "tol": 1e-8, "tuned": False,
                "shapes": rng.randrange(1 << 20)}
    if kind == "fills":
        return {"kind": "fills", "count": _log_uniform(rng, 1, 200), "ragged": True,
                "parent": rng.randint(48, 256), "ratio": rng.choice([1, 2, 4]), "shapes": rng.randrange(1 << 20)}
    if kind == "levels":
        return {"kind": "levels", "n": rng.choice([64, 80, 96, 112, 128]), "refinements": rng.randint(1, 8),
                "side": rng.choice([24, 32, 40, 48]), "prec": rng.choice(["fp64", "mixed"]), "alpha": 0.1,
                "tol": 1e-8, "tuned": False}
    if kind == "force":
        return {"kind": "force", "n0": _log_uniform(rng, 30, 400), "n1": _log_uniform(rng, 30, 320),
                "n2": _log_uniform(rng, 30, 256)}
    c = {"kind": kind, "lattice": _log_uniform(rng, 28, 250), "scheme": rng.choice(["cic", "tsc"]),
         "shuffled": rng.random() < 0.5}
    if kind == "assign":
        return dict(c, n0=_log_uniform(rng, 24, 256), n1=_log_uniform(rng, 24, 256), n2=_log_uniform(rng, 24, 256))
    return dict(c, n0=rng.randint(16, 96), n1=rng.randint(16, 96), n2=rng.randint(16, 96),
                box=rng.randint(128, 512))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7fffffff)


def _modes(n):
    """Integer wave numbers (kz, ky, kx), shaped to broadcast over an rfftn."""
    n0, n1, n2 = n
    opt = dict(dtype=torch.float64, device="cuda")
    return (torch.fft.fftfreq(n2, d=1.0 / n2, **opt)[:, None, None],
            torch.fft.fftfreq(n1, d=1.0 / n1, **opt)[None, :, None],
            torch.fft.rfftfreq(n0, d=1.0 / n0, **opt)[None, None, :])


def _gaussian(n, index, gen, kmax=None):
    """Unit-variance Gaussian random field with P(k) ~ k^index, cut at kmax."""
    n0, n1, n2 = n
    wk = torch.fft.rfftn(torch.randn((n2, n1, n0), generator=gen, dtype=torch.float64, device="cuda"))
    kz, ky, kx = _modes(n)
    m2 = kz * kz + ky * ky + kx * kx
    m2[0, 0, 0] = 1.0
    amp = m2.pow(0.25 * index)
    if kmax is not None:
        amp = torch.where(m2 <= kmax * kmax, amp, 0.0)
    amp[0, 0, 0] = 0.0
    g = torch.fft.irfftn(wk * amp, s=(n2, n1, n0))
    return g / g.std()


def _lognormal(n, sigma, gen):
    rho = torch.exp(sigma * _gaussian(n, -2.0, gen))
    d = rho / rho.mean() - 1.0
    return (d - d.mean()).contiguous()


def _tophat(n, gen):
    """Sphere of radius 0.1 and contrast 50 about a random centre, mean removed."""
    c = torch.rand(3, generator=gen, dtype=torch.float64, device="cuda")
    ax = [(torch.arange(m, dtype=torch.float64, device="cuda") + 0.5) / m for m in n]
    d = [torch.remainder(a - c[i] + 0.5, 1.0) - 0.5 for i, a in enumerate(ax)]
    r2 = d[2][:, None, None] ** 2 + d[1][None, :, None] ** 2 + d[0][None, None, :] ** 2
    t = torch.where(r2 < 0.01, 50.0, 0.0).to(torch.float64)
    return (t - t.mean()).contiguous()


def _potential(n, gen, amplitude):
    """Solution of the linear Poisson problem of a lognormal field, unit box."""
    d = _lognormal(n, 1.0, gen)
    kz, ky, kx = _modes(n)
    k2 = (2.0 * math.pi) ** 2 * (kz * kz + ky * ky + kx * kx)
    k2[0, 0, 0] = 1.0
    pk = -torch.fft.rfftn(d) / k2
    pk[0, 0, 0] = 0.0
    return (amplitude * torch.fft.irfftn(pk, s=tuple(reversed(n)))).contiguous()


def _particles(m, gen, shuffled=False):
    """m^3 lattice particles moved by a Zel'dovich displacement (linear spectrum
    k^-1.5 up to a quarter of the Nyquist frequency); rows of (x, y, z) in [0, 1)."""
    n = (m, m, m)
    dk = torch.fft.rfftn(_gaussian(n, -1.5, gen, kmax=0.125 * m))
    kz, ky, kx = (2.0 * math.pi * k for k in _modes(n))
    k2 = kz * kz + ky * ky + kx * kx
    k2[0, 0, 0] = 1.0
    q = (torch.arange(m, dtype=torch.float64, device="cuda") + 0.5) / m
    lattice = (q[None, None, :], q[None, :, None], q[:, None, None])
    pos = torch.empty((m, m, m, 3), dtype=torch.float64, device="cuda")
    for a, k in enumerate((kx, ky, kz)):
        psi = torch.fft.irfftn(1j * k * dk / k2, s=n)
        pos[..., a] = torch.remainder(lattice[a] + ZELDOVICH_AMPLITUDE * psi, 1.0)
    pos = pos.view(-1, 3)
    if shuffled:
        pos = pos[torch.randperm(pos.shape[0], generator=gen, device="cuda")]
    return pos.contiguous()


_tune_copy = None


def _flags(case):
    """Graph replay; tuned cases take the committed schedules, as the benchmark
    does, from a copy (the library appends what it tunes itself)."""
    global _tune_copy
    if not case["tuned"]:
        return vmg.GRAPH
    if _tune_copy is None:
        _tune_copy = os.path.join(tempfile.mkdtemp(prefix="vmg_tune_"), "tune.txt")
        shutil.copyfile(TUNE_FILE, _tune_copy)
        os.environ["VMG_TUNE_CACHE"] = _tune_copy
    return vmg.GRAPH | vmg.AUTOTUNE


def _patch_shapes(case):
    """Cells per axis of every patch: the sides in turn, or (ragged) each axis
    drawn on its own: c 2^k with c = 3..8 and one k per patch where the patch is
    solved (it has to coarsen), any size where it is only filled."""
    if not case["ragged"]:
        sides = [int(s) for s in case["sides"].split(",")]
        return [(sides[i % len(sides)],) * 3 for i in range(case["count"])]
    r = random.Random(case["shapes"])
    if case["kind"] == "fills":
        return [tuple(r.randint(9, 80) for _ in range(3)) for _ in range(case["count"])]
    out = []
    for _ in range(case["count"]):
        s = 1 << r.randint(2, 3)
        out.append(tuple(r.randint(3, 8) * s for _ in range(3)))
    return out


def _patch_layout(case, seed):
    """Grids and origins (on the refinement lattice) of the patches."""
    lattice = case["parent"] * case["ratio"]
    r = random.Random(int(seed))
    grids, origins, off, goff = [], [], 0, 0
    for n in _patch_shapes(case):
        grids.append(vmg.make_grid(n, 1.0 / lattice, vmg.DIRICHLET, off, goff))
        origins.append(tuple(r.randrange(lattice) for _ in range(3)))
        off += n[0] * n[1] * n[2]
        goff += vmg.ghost_count(n)
    return grids, origins, off, goff


def _densest(delta, count, apart):
    """`count` cells (x, y, z) of the highest density at least `apart` cells from
    one another along some axis (periodic)."""
    n = delta.shape[0]
    order = torch.argsort(delta.reshape(-1), descending=True)[:200000].cpu().tolist()
    found = []
    for e in order:
        c = (e % n, (e // n) % n, e // (n * n))
        if all(any(min((a - b) % n, (b - a) % n) >= apart for a, b in zip(c, o)) for o in found):
            found.append(c)
            if len(found) == count:
                return found
    return found + found[:count - len(found)]


def _levels_layout(case, pos):
    """Domain grid, a refinement over each of the densest cells, and a second-level
    refinement in the middle of each; every grid's density from the particles."""
    n, side, count = case["n"], case["side"], case["refinements"]
    mean = pos.shape[0] / n ** 3
    domain = vmg.mass_assign(pos, n, vmg.ASSIGN_CIC)
    grids, nests = [vmg.make_grid(n)], [vmg.make_nest(-1)]
    parts, off, goff = [domain.reshape(-1)], n ** 3, 0

    def add(parent, origin, h, corner):
        nonlocal off, goff
        grids.append(vmg.make_grid(side, h, vmg.DIRICHLET, off, goff))
        nests.append(vmg.make_nest(parent, origin))
        off += side ** 3
        goff += vmg.ghost_count(side)
        d = vmg.mass_assign_region(pos, side, h, corner, mean * (h * n) ** 3, vmg.ASSIGN_CIC)
        parts.append(d.reshape(-1))

    h1, h2 = 0.5 / n, 0.25 / n
    first = []
    for c in _densest(domain, count, side // 2 + 1):
        o = tuple((2 * v + 1 - side // 2) % (2 * n) for v in c)
        first.append(o)
        add(0, o, h1, [v * h1 for v in o])
    for k, o in enumerate(first):
        inner = (side // 2,) * 3
        add(1 + k, inner, h2, [((2 * o[a] + inner[a]) * h2) % 1.0 for a in range(3)])
    return grids, nests, torch.cat(parts).contiguous(), goff


def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    new = dict(dtype=torch.float64, device="cuda")
    if kind == "solve":
        n = (case["n0"], case["n1"], case["n2"])
        if case["field"] == "tophat":
            delta = _tophat(n, gen)
        elif case["field"] == "zeldovich":
            delta = vmg.mass_assign(_particles(n[0], gen), n, vmg.ASSIGN_CIC)
        else:
            delta = _lognormal(n, case["sigma"], gen)
        st = {"case": case, "delta": delta}
        if case["kept"]:
            params = vmg.make_params(case["alpha"], KAPPA, case["tol"], 60, PRECISIONS[case["prec"]],
                                     flags=_flags(case))
            st["plan"] = vmg.Plan([vmg.make_grid(n)], params)
            st["phi"] = torch.zeros_like(delta)
        return st
    if kind in ("patches", "fills"):
        grids, origins, cells, ghosts = _patch_layout(case, seed)
        parent = _potential((case["parent"],) * 3, gen, 0.5)
        st = {"case": case, "grids": grids, "origins": origins, "parent": parent, "parent_h": 1.0 / case["parent"],
              "ghost": torch.zeros(ghosts, **new), "phi": torch.zeros(cells, **new)}
        if kind == "patches":
            vmg.fill_ghosts(parent, st["parent_h"], grids, origins, st["ghost"])
            vmg.fill_interior(parent, st["parent_h"], grids, origins, st["phi"])
            st["guess"] = st["phi"].clone()
            st["delta"] = torch.cat([_lognormal(tuple(g.n), case["sigma"], gen).reshape(-1) for g in grids])
            params = vmg.make_params(case["alpha"], KAPPA, case["tol"], 60, PRECISIONS[case["prec"]],
                                     flags=_flags(case))
            st["plan"] = vmg.Plan(grids, params)
        return st
    if kind == "levels":
        pos = _particles(case["n"], gen)
        grids, nests, delta, ghosts = _levels_layout(case, pos)
        params = vmg.make_params(case["alpha"], KAPPA, case["tol"], 60, PRECISIONS[case["prec"]], flags=_flags(case))
        return {"case": case, "plan": vmg.LevelsPlan(grids, nests, params), "delta": delta,
                "ghost": torch.zeros(ghosts, **new), "phi": torch.zeros_like(delta)}
    n = (case["n0"], case["n1"], case["n2"])
    if kind == "force":
        return {"case": case, "newton": _potential(n, gen, 1.0), "phi": _potential(n, gen, 0.3),
                "psi": torch.empty(n[::-1], **new), "force": torch.empty((3,) + n[::-1], **new)}
    pos = _particles(case["lattice"], gen, case["shuffled"])
    need = vmg.mass_assign_workspace(pos.shape[0], n)
    st = {"case": case, "pos": pos, "delta": torch.empty(n[::-1], **new),
          "workspace": torch.empty(need, dtype=torch.uint8, device="cuda")}
    if kind == "region":
        r = random.Random(int(seed))
        st["corner"] = [r.randrange(case["box"]) / case["box"] for _ in range(3)]
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        if not case["kept"]:
            phi, info = vmg.solve_field(state["delta"], case["alpha"], KAPPA, case["tol"], PRECISIONS[case["prec"]])
        else:
            phi = state["phi"].zero_()
            info = state["plan"].solve(state["delta"], phi, allow_noconv=True)[0]
        return {"phi": phi, "cbar": info["compat_c"], "cycles": info["cycles"]}
    if kind == "patches":
        phi = state["phi"].copy_(state["guess"])
        info = state["plan"].solve(state["delta"], phi, ghost=state["ghost"], allow_noconv=True)
        return {"phi": phi, "cycles": info[0]["cycles"]}
    if kind == "fills":
        vmg.fill_ghosts(state["parent"], state["parent_h"], state["grids"], state["origins"], state["ghost"])
        vmg.fill_interior(state["parent"], state["parent_h"], state["grids"], state["origins"], state["phi"])
        return {"ghost": state["ghost"], "phi": state["phi"]}
    if kind == "levels":
        phi = state["phi"].zero_()
        info = state["plan"].solve(state["delta"], state["ghost"], phi, allow_noconv=True)
        return {"phi": phi, "ghost": state["ghost"], "cycles": [r["cycles"] for r in info[:1] + info[-1:]]}
    if kind == "force":
        psi, force = vmg.total_force(state["newton"], state["phi"], 1.0 / case["n0"], state["psi"], state["force"])
        return {"psi": psi, "force": force}
    n = (case["n0"], case["n1"], case["n2"])
    scheme = SCHEMES[case["scheme"]]
    if kind == "assign":
        return vmg.mass_assign(state["pos"], n, scheme, state["delta"], state["workspace"])
    h = 1.0 / case["box"]
    return vmg.mass_assign_region(state["pos"], n, h, state["corner"], state["pos"].shape[0] * h ** 3, scheme,
                                  state["delta"], state["workspace"])


def work(case):
    """Bytes: every input read once, every output written once.  Operations: one
    evaluation of the discrete equation per cell for a solve (the iteration needs
    several; how many is not fixed by the problem)."""
    kind = case["kind"]
    if kind in ("patches", "fills"):
        shapes = _patch_shapes(case)
        cells = sum(a * b * c for a, b, c in shapes)
        ghosts = sum(2 * (b * c + a * c + a * b) + 4 * (a + b + c) for a, b, c in shapes)
        if kind == "patches":
            return {"bytes": 24 * cells + 8 * ghosts, "flops": 70 * cells}
        parent = min(case["parent"] ** 3, (cells + ghosts) / case["ratio"] ** 3)
        return {"bytes": 8 * (cells + ghosts + parent), "flops": 14 * (cells + ghosts)}
    if kind == "levels":
        cells = case["n"] ** 3 + 2 * case["refinements"] * case["side"] ** 3
        return {"bytes": 24 * cells, "flops": 70 * cells}
    cells = case["n0"] * case["n1"] * case["n2"]
    if kind == "solve":
        return {"bytes": 24 * cells, "flops": 70 * cells}
    if kind == "force":
        return {"bytes": 48 * cells, "flops": 8 * cells}
    particles = case["lattice"] ** 3
    # a region is reached by the particles of its own volume; each particle's
    # position has to be read to know
    inside = particles if kind == "assign" else particles * cells / case["box"] ** 3
    per = 27 if case["scheme"] == "tsc" else 8
    return {"bytes": 24 * particles + 8 * cells, "flops": 10 * particles + (2 * per + 20) * inside}


# ---------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# ---------------------------------------------------------------------------
def _weights(u, scheme):
    """First stencil cell and the weights along one axis; u in cells."""
    if scheme == "cic":
        g = torch.floor(u - 0.5)
        t = u - 0.5 - g
        return g.long(), [1.0 - t, t]
    c = torch.floor(u)
    d = u - c - 0.5
    return c.long() - 1, [0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2]


def _exact_deposit(case, st):
    n = (case["n0"], case["n1"], case["n2"])
    pos, region = st["pos"], case["kind"] == "region"
    axes = []
    for a in range(3):
        x = pos[:, a]
        if region:
            h = 1.0 / case["box"]
            off = torch.remainder(x - st["corner"][a], 1.0)
            off = torch.where(off > (n[a] + 2) * h, off - 1.0, off)
            axes.append(_weights(off / h, case["scheme"]))
        else:
            axes.append(_weights(torch.remainder(x, 1.0) * n[a], case["scheme"]))
    rho = torch.zeros(n[0] * n[1] * n[2], dtype=torch.float64, device=pos.device)
    (cx, wx), (cy, wy), (cz, wz) = axes
    for k, wk in enumerate(wz):
        for j, wj in enumerate(wy):
            for i, wi in enumerate(wx):
                cell = [cx + i, cy + j, cz + k]
                w = wi * wj * wk
                if region:
                    inside = torch.ones_like(w, dtype=torch.bool)
                    for a in range(3):
                        inside &= (cell[a] >= 0) & (cell[a] < n[a])
                    w = torch.where(inside, w, 0.0)
                idx = [torch.remainder(cell[a], n[a]) for a in range(3)]
                rho.index_add_(0, (idx[2] * n[1] + idx[1]) * n[0] + idx[0], w)
    mean = pos.shape[0] / case["box"] ** 3 if region else pos.shape[0] / (n[0] * n[1] * n[2])
    return (rho / mean - 1.0).view(n[::-1])


def _ghost_cells(n):
    """Coordinates of the ghost values in their compact order (see vmg.h)."""
    n0, n1, n2 = n
    out = []

    def block(fixed, slow, fast):
        """Values at the two axes `slow`, `fast` (None: edge) with the others fixed."""
        c = [None] * 3
        s = torch.arange(n[slow]) if slow is not None else torch.zeros(1, dtype=torch.long)
        f = torch.arange(n[fast])
        grid = torch.cartesian_prod(s, f)
        if slow is not None:
            c[slow] = grid[:, 0]
        c[fast] = grid[:, 1]
        for a, v in fixed.items():
            c[a] = torch.full((grid.shape[0],), v, dtype=torch.long)
        out.append(torch.stack(c, 1))

    for x in (-1, n0):
        block({0: x}, 2, 1)
    for y in (-1, n1):
        block({1: y}, 2, 0)
    for z in (-1, n2):
        block({2: z}, 1, 0)
    for z in (-1, n2):
        for y in (-1, n1):
            block({1: y, 2: z}, None, 0)
    for z in (-1, n2):
        for x in (-1, n0):
            block({0: x, 2: z}, None, 1)
    for y in (-1, n1):
        for x in (-1, n0):
            block({0: x, 1: y}, None, 2)
    return torch.cat(out)


def _exact_fill(st, g, origin, cells):
    parent, np_ = st["parent"], st["parent"].shape[0]
    lo, fr = [], []
    for a in range(3):
        u = (origin[a] + cells[:, a].double() + 0.5) * (g.h / st["parent_h"]) - 0.5
        lo.append(torch.floor(u).long())
        fr.append(u - torch.floor(u))
    v = 0.0
    for c in range(8):
        d = [(c >> a) & 1 for a in range(3)]
        w = 1.0
        for a in range(3):
            w = w * (fr[a] if d[a] else 1.0 - fr[a])
        i = [torch.remainder(lo[a] + d[a], np_) for a in range(3)]
        v = v + w * parent[i[2], i[1], i[0]]
    return v


def exact(case, seed):
    """None for the solves: they return the state their stopping rule ends at, which
    is a tolerance away from the discrete solution."""
    kind = case["kind"]
    if kind not in ("assign", "region", "force", "fills"):
        return None
    st = prepare(case, seed)
    if kind in ("assign", "region"):
        return _exact_deposit(case, st)
    if kind == "force":
        psi = st["newton"] + 0.5 * st["phi"]
        h = 1.0 / case["n0"]
        return {"psi": psi, "force": torch.stack([(torch.roll(psi, 1, d) - torch.roll(psi, -1, d)) / (2.0 * h)
                                                  for d in (2, 1, 0)])}
    dev = st["parent"].device
    ghost, phi = [], []
    for g, o in zip(st["grids"], st["origins"]):
        n = tuple(g.n)
        ghost.append(_exact_fill(st, g, o, _ghost_cells(n).to(dev)))
        z, y, x = (torch.arange(m) for m in n[::-1])
        zyx = torch.cartesian_prod(z, y, x)
        phi.append(_exact_fill(st, g, o, zyx.flip(1).to(dev)))
    return {"ghost": torch.cat(ghost), "phi": torch.cat(phi)}
