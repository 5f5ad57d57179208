"""What is timed on this library: calls of its public entry points over the
sizes, particle sets and options that programs use it with.

Every case is one pass of such a program: a density + force pass on kept cells
(``Context.pass_``), a new snapshot (``Context.build_cells`` and then density
and force), a leapfrog step (``Context.step``), or the near-field gravity
(``Context.gravity_p2p``). The particle sets follow the repository's own
workloads (jittered lattices, one box or many, the Sedov-like blast, Plummer
spheres on a uniform background, a log-normal density field), drawn on the GPU
from a seed.

``exact`` recomputes a pass in 64 bits with plain torch: a neighbour search of
its own, h solved to the root, and the force formulas of ``include/sph.h``.
"""

import math

import torch

import paper_1508_00115_amd as sph

DEV = "cuda"
N_NGB, GAMMA, ALPHA = 48.0, 5.0 / 3.0, 0.8
GRAV_EPS, COURANT = 1e-3, 0.2

# Context keywords a case may carry.
PARAMS = ("h_margin", "cell_ratio", "leaf_target", "schedule", "tile_cap", "cell_order", "balsara",
          "signal_velocity")

# The cell parameters stored with the library for the sets they were tuned on.
TUNED_BOXES = {"h_margin": 1.05, "cell_ratio": 1.0, "leaf_target": 32, "schedule": 1, "tile_cap": 128,
               "cell_order": 1}
TUNED_BLAST = {"h_margin": 1.05, "cell_ratio": 0.5, "leaf_target": 64, "schedule": 0, "tile_cap": 128,
               "cell_order": 2}
TUNED_FIELD = {"h_margin": 1.05, "cell_ratio": 0.5, "leaf_target": 64, "schedule": 0, "tile_cap": 128,
               "cell_order": 1}


def listed():
    return [
        # one small box with the library's defaults: a unit test, a toy run, an
        # interactive call; launches and the host round trip decide
        {"name": "pass_small_16", "call": "pass", "set": "lattice", "boxes": 1, "side_min": 16, "side_max": 16,
         "jitter": 0.1, "vel": 0.1},
        # a few boxes of odd sizes with the defaults: a small ensemble
        {"name": "pass_boxes_odd", "call": "pass", "set": "lattice", "boxes": 7, "side_min": 11, "side_max": 27,
         "jitter": 0.2, "vel": 0.1},
        # the Sedov-like blast at its start, tuned parameters
        {"name": "pass_sedov_64", "call": "pass", "set": "blast", "boxes": 1, "side_min": 64, "side_max": 64,
         "jitter": 0.1, "vel": 0.0, **TUNED_BLAST},
        # the throughput workload: 256 boxes in one captured pass, tuned parameters
        {"name": "pass_boxes_256", "call": "pass", "set": "lattice", "boxes": 256, "side_min": 20, "side_max": 40,
         "jitter": 0.1, "vel": 0.1, **TUNED_BOXES},
        # clustered matter: adaptive cells, smoothing lengths over a factor of 30
        {"name": "pass_clustered_1m", "call": "pass", "set": "spheres", "background": 1 << 19, "spheres": 64,
         "per_sphere": 8192, **TUNED_BLAST},
        # the largest set: a log-normal field of 2^24 particles, deep trees
        {"name": "pass_lognormal_256", "call": "pass", "set": "lognormal", "mesh": 256, "sigma": 1.5,
         **TUNED_FIELD},
        # particles of unequal masses (several resolutions in one box), an odd side
        {"name": "pass_mixed_41", "call": "pass", "set": "lattice", "boxes": 1, "side_min": 41, "side_max": 41,
         "jitter": 0.3, "vel": 0.2, "mass_spread": 0.5},
        # the viscosity limiter and the signal velocities a simulation would switch on
        {"name": "pass_balsara_64", "call": "pass", "set": "lattice", "boxes": 64, "side_min": 20, "side_max": 40,
         "jitter": 0.2, "vel": 0.1, "balsara": 1, "signal_velocity": 1},
        # snapshots analysed one after another: new cells, then density and force as
        # separate calls, defaults
        {"name": "snapshot_lattice_64", "call": "snapshot", "set": "lattice", "boxes": 1, "side_min": 64,
         "side_max": 64, "jitter": 0.2, "vel": 0.1},
        {"name": "snapshot_clustered_1m", "call": "snapshot", "set": "spheres", "background": 1 << 19,
         "spheres": 64, "per_sphere": 8192},
        # time integration: the Courant step and one kick-drift-kick step, cells kept or rebuilt
        {"name": "step_48", "call": "step", "set": "lattice", "boxes": 1, "side_min": 48, "side_max": 48,
         "jitter": 0.2, "vel": 0.2, "signal_velocity": 1},
        # the near-field gravity over the same cells
        {"name": "gravity_boxes_256", "call": "gravity", "set": "lattice", "boxes": 256, "side_min": 20,
         "side_max": 40, "jitter": 0.1, "vel": 0.0, **TUNED_BOXES},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges the listed ones span: any call, set and parameters."""
    c = {"call": rng.choice(["pass", "pass", "pass", "snapshot", "step", "gravity"])}
    c["set"] = rng.choice(["lattice", "lattice", "blast", "spheres", "lognormal"])
    if c["set"] in ("lattice", "blast"):
        c["boxes"] = 1 if c["set"] == "blast" or rng.random() < 0.4 else _log_int(rng, 2, 128)
        top = 100 if c["boxes"] == 1 else 40
        a, b = _log_int(rng, 10, top), _log_int(rng, 10, top)
        c["side_min"], c["side_max"] = (min(a, b), max(a, b)) if c["boxes"] > 1 else (a, a)
        c["jitter"] = round(rng.uniform(0.05, 0.4), 3)
        c["vel"] = round(rng.uniform(0.02, 0.3), 3)
        if rng.random() < 0.2:
            c["mass_spread"] = 0.5
    elif c["set"] == "spheres":
        c["spheres"] = _log_int(rng, 2, 64)
        c["per_sphere"] = _log_int(rng, 500, 8192)
        # the background holds about half the particles, as in the listed set
        c["background"] = int(c["spheres"] * c["per_sphere"] * rng.uniform(0.8, 2.0)) + 8192
    else:
        c["mesh"] = _log_int(rng, 40, 128)
        # (the emptiest cells' smoothing lengths have to stay below a third of the box)
        c["sigma"] = round(rng.uniform(0.5, min(1.5, 0.55 * math.log(0.1 * c["mesh"]))), 3)
    c["h_margin"] = rng.choice([1.05, 1.1, 1.18, 1.26])
    c["cell_ratio"] = rng.choice([0.5, 1.0])
    c["leaf_target"] = rng.choice([32, 64])
    c["schedule"] = rng.choice([0, 1])
    c["tile_cap"] = rng.choice([128, 512])
    c["cell_order"] = rng.choice([0, 1, 2])
    if c["call"] == "step":
        c["signal_velocity"] = 1
    elif c["call"] == "pass" and rng.random() < 0.25:
        c["balsara"] = c["signal_velocity"] = 1
    return c


# ---- inputs -----------------------------------------------------------------------------


def _sides(case):
    """Sides of the boxes: particle counts spread over [side_min^3, side_max^3] on
    their logarithm (a golden-ratio sequence), the same for every seed."""
    lo, hi = case["side_min"], case["side_max"]
    if case["boxes"] == 1:
        return [lo]
    return [min(hi, max(lo, int(round(lo * (hi / lo) ** ((0.5 + b * 0.6180339887498949) % 1.0)))))
            for b in range(case["boxes"])]


def _count(case):
    if case["set"] in ("lattice", "blast"):
        return sum(s ** 3 for s in _sides(case))
    if case["set"] == "spheres":
        return case["background"] + case["spheres"] * case["per_sphere"]
    return case["mesh"] ** 3


def _guess(mass, rho):
    """h of a sphere that holds N_NGB particles of this mass at density rho."""
    return (3.0 * N_NGB * mass / (4.0 * math.pi * rho)) ** (1.0 / 3.0)


def _lattice(case, g):
    pos, vel, mass, u, h0, first = [], [], [], [], [], [0]
    f64 = dict(dtype=torch.float64, device=DEV)
    for s in _sides(case):
        n = s ** 3
        x = (torch.arange(s, **f64) + 0.5) / s
        p = torch.stack(torch.meshgrid(x, x, x, indexing="ij"), dim=-1).reshape(n, 3)
        p = p + (torch.rand((n, 3), generator=g, **f64) * 2.0 - 1.0) * (case["jitter"] / s)
        pos.append(p - torch.floor(p))
        vel.append(torch.randn((n, 3), generator=g, device=DEV) * case["vel"])
        m = torch.full((n,), 1.0 / n, **f64)
        spread = case.get("mass_spread", 0.0)
        if spread:
            m = m * (1.0 + spread * (torch.rand(n, generator=g, **f64) * 2.0 - 1.0))
        mass.append(m)
        e = torch.ones(n, device=DEV)
        if case["set"] == "blast":
            e = e * 1e-5
            r2 = ((pos[-1] - 0.5) ** 2).sum(1)
            e[torch.sort(r2, stable=True)[1][:32]] = n / 32.0
        u.append(e)
        h0.append(torch.full((n,), _guess(1.0 / n, 1.0), **f64))
        first.append(first[-1] + n)
    cat = torch.cat
    return cat(pos), cat(vel), cat(mass), cat(u), cat(h0), first


def _spheres(case, g):
    f64 = dict(dtype=torch.float64, device=DEV)
    nb, ns, per = case["background"], case["spheres"], case["per_sphere"]
    n = nb + ns * per
    centre = torch.rand((ns, 3), generator=g, **f64)
    scale = torch.exp(math.log(0.005) + torch.rand(ns, generator=g, **f64) * math.log(10.0))
    # Plummer radii below half the box, by inverting the cumulative profile up to there
    top = (1.0 + (scale / 0.5) ** 2) ** -1.5
    x = torch.rand((ns, per), generator=g, **f64).clamp_min(1e-12) * top[:, None]
    r = scale[:, None] / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
    d = torch.randn((ns, per, 3), generator=g, **f64)
    d = d / d.norm(dim=2, keepdim=True)
    pos = torch.cat([torch.rand((nb, 3), generator=g, **f64),
                     (centre[:, None] + r[..., None] * d).reshape(-1, 3)])
    pos = pos - torch.floor(pos)
    rho = torch.full((n,), nb / n, **f64)
    for k in range(ns):
        dx = pos - centre[k]
        dx = dx - torch.round(dx)
        a2 = float(scale[k]) ** 2
        rho += per / n * 3.0 / (4.0 * math.pi * a2 ** 1.5) * (1.0 + (dx * dx).sum(1) / a2) ** -2.5
    vel = torch.randn((n, 3), generator=g, device=DEV) * 0.1
    return (pos, vel, torch.full((n,), 1.0 / n, **f64), torch.ones(n, device=DEV), _guess(1.0 / n, rho), [0, n])


def _lognormal(case, g):
    f64 = dict(dtype=torch.float64, device=DEV)
    m = case["mesh"]
    n = m ** 3
    k1, k3 = torch.fft.fftfreq(m, **f64) * m, torch.fft.rfftfreq(m, **f64) * m
    k2 = k1[:, None, None] ** 2 + k1[None, :, None] ** 2 + k3[None, None, :] ** 2
    k2[0, 0, 0] = 1.0
    dk = torch.fft.rfftn(torch.randn((m, m, m), generator=g, **f64)) / torch.sqrt(k2)  # P(k) ~ k^-2
    dk[0, 0, 0] = 0.0
    delta = torch.fft.irfftn(dk, s=(m, m, m))
    rho = torch.exp(delta * (case["sigma"] / delta.std()))
    rho = (rho / rho.mean()).reshape(-1)
    # particles per mesh cell in whole numbers, so that the sums are exact
    edges = torch.cumsum((rho * 2.0 ** 24).to(torch.int64) + 1, 0)
    x = (torch.rand(n, generator=g, **f64) * edges[-1].double()).to(torch.int64)
    cell = torch.sort(torch.searchsorted(edges, x, right=True).clamp_max(n - 1))[0]
    ijk = torch.stack([cell // (m * m), (cell // m) % m, cell % m], dim=1)
    pos = (ijk + torch.rand((n, 3), generator=g, **f64)) / m
    pos = pos - torch.floor(pos)
    vel = torch.empty((n, 3), **f64)
    for ax, kv in enumerate((k1[:, None, None], k1[None, :, None], k3[None, None, :])):
        vf = torch.fft.irfftn(1j * kv * dk / k2, s=(m, m, m))
        vel[:, ax] = (vf * (0.1 / vf.std())).reshape(-1)[cell]
    return (pos, vel, torch.full((n,), 1.0 / n, **f64), torch.ones(n, device=DEV), _guess(1.0 / n, rho[cell]),
            [0, n])


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    make = {"lattice": _lattice, "blast": _lattice, "spheres": _spheres, "lognormal": _lognormal}[case["set"]]
    pos, vel, mass, u, h0, first = make(case, g)
    f = torch.float32
    return {"pos": pos.contiguous(), "vel": vel.to(f).contiguous(), "mass": mass.to(f), "u": u.to(f),
            "h0": h0.to(f), "first": first}


def _cutoff(h0):
    return 0.95 * float(h0.min())


# ---- the calls --------------------------------------------------------------------------


def prepare(case, seed):
    """The particles on the GPU, the context with its cells (a snapshot builds
    them in the call) and the output buffers a program keeps."""
    s = _inputs(case, seed)
    n = s["pos"].shape[0]
    s["call"] = case["call"]
    s["balsara"] = bool(case.get("balsara", 0))
    s["h"] = s["h0"].clone()
    s["rho"], s["f"], s["dudt"] = (torch.empty(n, device=DEV) for _ in range(3))
    s["acc"] = torch.empty((n, 3), device=DEV)
    ctx = sph.Context(0, **{k: case[k] for k in PARAMS if k in case})
    s["ctx"] = ctx
    if case["call"] != "snapshot":
        ctx.build_cells(s["pos"], s["h0"], s["first"], [1.0] * (len(s["first"]) - 1))
    if case["call"] == "step":
        # a simulation under way: the rates at the start of its first step
        ctx.pass_(s["mass"], s["h"], s["vel"], s["u"], rho=s["rho"], f=s["f"], acc=s["acc"], dudt=s["dudt"])
    if case["call"] == "gravity":
        s["r_cut"] = _cutoff(s["h0"])
    return s


def run(s):
    ctx = s["ctx"]
    if s["call"] == "pass":
        s["h"].copy_(s["h0"])  # every pass solves h from the guesses
        ctx.pass_(s["mass"], s["h"], s["vel"], s["u"], rho=s["rho"], f=s["f"], acc=s["acc"], dudt=s["dudt"])
        out = {k: s[k] for k in ("h", "rho", "f", "acc", "dudt")}
        if s["balsara"]:
            out["balsara"] = ctx.balsara()
        return out
    if s["call"] == "snapshot":
        s["h"].copy_(s["h0"])
        ctx.build_cells(s["pos"], s["h0"], s["first"], [1.0] * (len(s["first"]) - 1))
        ctx.density(s["mass"], s["h"], rho=s["rho"], f=s["f"])
        ctx.force(s["vel"], s["u"], acc=s["acc"], dudt=s["dudt"])
        return {k: s[k] for k in ("h", "rho", "f", "acc", "dudt")}
    if s["call"] == "step":
        dt = ctx.timestep(COURANT)
        ctx.step(dt, s["pos"], s["mass"], s["h"], s["vel"], s["u"], s["acc"], s["dudt"], rho=s["rho"], f=s["f"])
        return {k: s[k] for k in ("pos", "vel", "u", "h", "rho", "f", "acc", "dudt")}
    ctx.gravity_p2p(s["mass"], 1.0, GRAV_EPS, s["r_cut"], acc=s["acc"])
    return {"acc": s["acc"]}


def work(case):
    """Bytes: each particle's inputs once (FP32 offsets or FP64 positions, m, h, v,
    u) and its outputs once. Operations: 45 neighbours inside h at the first and
    at the last trial h (26 each), 47 force pairs (61 each, both sides), 22
    pairs inside the gravity cutoff (22 each)."""
    n = _count(case)
    pair = 2 * 45 * 26 + 47 * 61
    if case["call"] == "gravity":
        return {"bytes": n * (16 + 4 + 12), "flops": n * 22 * 22}
    if case["call"] == "snapshot":
        return {"bytes": n * (24 + 4 + 4 + 12 + 4 + 28), "flops": n * pair}
    if case["call"] == "step":
        # positions, v, u, a, du/dt and h read and written; m, rho, f
        return {"bytes": n * (2 * (24 + 12 + 4 + 12 + 4 + 4) + 4 + 8), "flops": n * pair}
    extra = 47 * 40 if case.get("balsara") else 0
    return {"bytes": n * (16 + 4 + 4 + 12 + 4 + 28), "flops": n * (pair + extra)}


# ---- the same in 64 bits ------------------------------------------------------------------


def _pairs(pos, R, budget=30_000_000):
    """Ordered pairs (i, j) with r_ij < R_i (j = i among them) in the periodic
    unit box, in pieces: the query particles of the piece, the row of each pair
    among them, j and the separation. Queries are grouped by radius, each group
    on a grid of cells at least that wide."""
    n = pos.shape[0]
    r_top = float(R.max())
    lev = torch.floor(torch.log2(r_top / R)).clamp(0, 20).to(torch.int64)
    o = torch.tensor([[a, b, c] for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)], device=DEV)
    for lv in torch.unique(lev).tolist():
        ask = torch.nonzero(lev == lv)[:, 0]
        G = int(1.0 / (r_top / 2 ** lv))
        assert G >= 3, "a search radius above a third of the box"
        G = min(G, 400)
        c = torch.floor(pos * G).to(torch.int64).clamp_(0, G - 1)
        key = (c[:, 0] * G + c[:, 1]) * G + c[:, 2]
        order = torch.argsort(key)
        count = torch.bincount(key, minlength=G ** 3)
        start = torch.cumsum(count, 0) - count
        ask = ask[torch.argsort(key[ask])]
        for blk in torch.split(ask, 1_000_000):
            nb = (c[blk][:, None, :] + o[None]) % G
            nk = (nb[..., 0] * G + nb[..., 1]) * G + nb[..., 2]
            cnt = count[nk]
            tot = torch.cumsum(cnt.sum(1), 0)
            cut, a = [], 0
            while a < len(blk):
                base = 0 if a == 0 else int(tot[a - 1])
                b = max(a + 1, int(torch.searchsorted(tot, base + budget, right=True)))
                cut.append((a, min(b, len(blk))))
                a = b
            for a, b in cut:
                k, m = nk[a:b].reshape(-1), cnt[a:b].reshape(-1)
                slot = torch.repeat_interleave(torch.arange(len(k), device=DEV), m)
                within = torch.arange(len(slot), device=DEV) - (torch.cumsum(m, 0) - m)[slot]
                j = order[start[k][slot] + within]
                row = slot // 27
                q = blk[a:b]
                d = pos[q][row] - pos[j]
                d = d - torch.round(d)
                keep = (d * d).sum(1) < (R[q] ** 2)[row]
                yield q, row[keep], j[keep], d[keep]


def _w(q):
    return torch.where(q < 0.5, 1.0 - 6.0 * q * q * (1.0 - q), 2.0 * (1.0 - q).clamp_min(0.0) ** 3)


def _dw(q):
    return torch.where(q < 0.5, q * (18.0 * q - 12.0), -6.0 * (1.0 - q).clamp_min(0.0) ** 2)


def _rows(row, value, Q, fill):
    """The pairs' values as one padded row for each query."""
    cnt = torch.bincount(row, minlength=Q)
    out = torch.full((Q, int(cnt.max())), fill, dtype=torch.float64, device=DEV)
    out[row, torch.arange(len(row), device=DEV) - (torch.cumsum(cnt, 0) - cnt)[row]] = value
    return out


def _density64(pos, mass, h0):
    """h (the root of sum w(r / h) = 3 N_NGB / 32), rho and f of every particle."""
    n, target = pos.shape[0], 3.0 * N_NGB / 32.0
    h, rho, f = (torch.zeros(n, dtype=torch.float64, device=DEV) for _ in range(3))
    todo, R = torch.arange(n, device=DEV), 1.15 * h0
    while len(todo):
        mask = torch.zeros(n, dtype=torch.float64, device=DEV)
        mask[todo] = R[todo]
        short = []
        for q, row, j, d in _pairs_of(pos, mask, todo):
            r = _rows(row, d.norm(dim=1), len(q), 1e9)
            mj = _rows(row, mass[j], len(q), 0.0)
            top = R[q]
            few = _w(r / top[:, None]).sum(1) < target
            short.append(q[few])
            lo, hi, x = torch.zeros_like(top), top.clone(), torch.minimum(h0[q], top)
            for _ in range(60):
                t = r / x[:, None]
                S0, S1 = _w(t).sum(1), (t * _dw(t)).sum(1)
                below = S0 < target
                lo, hi = torch.where(below, x, lo), torch.where(below, hi, x)
                nx = x * torch.exp(-torch.log(S0 / target) * S0 / (-S1).clamp_min(1e-300))
                nx = torch.where((nx > lo) & (nx < hi), nx, 0.5 * (lo + hi))
                move = ((nx - x).abs() / x)[~few]
                x = nx
                if len(move) == 0 or float(move.max()) < 1e-15:
                    break
            t = r / x[:, None]
            M0, M1 = (mj * _w(t)).sum(1), (mj * t * _dw(t)).sum(1)
            h[q], rho[q] = x, 8.0 / math.pi * M0 / x ** 3
            f[q] = torch.where(M1 < 0.0, -3.0 * M0 / M1, torch.ones_like(M0))
        todo = torch.cat(short)
        R[todo] = (1.15 * R[todo]).clamp_max(1.0 / 3.0001)
    return h, rho, f


def _pairs_of(pos, R, todo):
    """_pairs for the particles of `todo` alone."""
    if len(todo) == pos.shape[0]:
        yield from _pairs(pos, R)
        return
    # a query set: the others get a radius too small to find more than themselves
    tiny = float(R[todo].min()) * 0.5 ** 19
    sel = torch.zeros(pos.shape[0], dtype=torch.bool, device=DEV)
    sel[todo] = True
    for q, row, j, d in _pairs(pos, torch.where(sel, R, torch.full_like(R, tiny))):
        if bool(sel[q].any()):
            keep = sel[q]
            new = torch.cumsum(keep, 0) - 1
            p = keep[row]
            yield q[keep], new[row[p]], j[p], d[p]


def _force64(pos, vel, mass, u, h, rho, f, balsara=False):
    """Accelerations, du/dt, Balsara factors and signal velocities."""
    n = pos.shape[0]
    z = lambda: torch.zeros(n, dtype=torch.float64, device=DEV)  # noqa: E731
    P = (GAMMA - 1.0) * rho * u
    c = torch.sqrt(GAMMA * (GAMMA - 1.0) * u)
    phi = f * P / rho ** 2
    B = None
    if balsara:
        div, curl = z(), [z(), z(), z()]
        for q, row, j, d in _pairs(pos, h):
            i = q[row]
            k = i != j
            i, j, d = i[k], j[k], d[k]
            r = d.norm(dim=1)
            mD = mass[j] * 8.0 / math.pi / h[i] ** 4 * _dw(r / h[i]) / r
            w = vel[i] - vel[j]
            div.index_add_(0, i, -mD * (w * d).sum(1))
            x = torch.linalg.cross(w, d)
            for a in range(3):
                curl[a].index_add_(0, i, mD * x[:, a])
        ad = div.abs() / rho
        den = ad + torch.sqrt(curl[0] ** 2 + curl[1] ** 2 + curl[2] ** 2) / rho + 1e-4 * c / h
        B = torch.where(den > 0, ad / den, torch.zeros_like(den))
    acc, du, vs = [z(), z(), z()], z(), c.clone()
    for q, row, j, d in _pairs(pos, h):
        i = q[row]
        r = d.norm(dim=1)
        k = r > 0
        i, j, d, r = i[k], j[k], d[k], r[k]
        Di = 8.0 / math.pi / h[i] ** 4 * _dw(r / h[i])
        Dj = torch.where(r < h[j], 8.0 / math.pi / h[j] ** 4 * _dw(r / h[j]), torch.zeros_like(r))
        vr = ((vel[i] - vel[j]) * d).sum(1) / r
        w = vr.clamp_max(0.0)
        sig = c[i] + c[j] - 3.0 * w
        pi = -ALPHA * sig * w / (rho[i] + rho[j])
        if B is not None:
            pi = pi * 0.5 * (B[i] + B[j])
        Db = 0.5 * (Di + Dj)
        G = phi[i] * Di + phi[j] * Dj + pi * Db
        far = r >= h[j]  # j does not find i inside its own h: its side of the pair is added here
        jf, i_f = j[far], i[far]
        for a in range(3):
            t = G * d[:, a] / r
            acc[a].index_add_(0, i, -mass[j] * t)
            acc[a].index_add_(0, jf, (mass[i] * t)[far])
        du.index_add_(0, i, mass[j] * (phi[i] * Di + 0.5 * pi * Db) * vr)
        du.index_add_(0, jf, (mass[i] * (phi[j] * Dj + 0.5 * pi * Db) * vr)[far])
        vs.scatter_reduce_(0, i, sig, "amax")
        vs.scatter_reduce_(0, jf, sig[far], "amax")
    return torch.stack(acc, dim=1), du, B, vs


def _gravity64(pos, mass, r_cut):
    n = pos.shape[0]
    acc = [torch.zeros(n, dtype=torch.float64, device=DEV) for _ in range(3)]
    for q, row, j, d in _pairs(pos, torch.full((n,), r_cut, dtype=torch.float64, device=DEV)):
        r2 = (d * d).sum(1)
        t = -mass[j] * (1.0 - r2 / r_cut ** 2) ** 2 * (r2 + GRAV_EPS ** 2) ** -1.5
        for a in range(3):
            acc[a].index_add_(0, q[row], t * d[:, a])
    return torch.stack(acc, dim=1)


def exact(case, seed):
    if _count(case) > 8_000_000:
        return None  # (minutes in plain torch)
    s = _inputs(case, seed)
    D = {k: s[k].double() for k in ("pos", "vel", "mass", "u", "h0")}
    r_cut = _cutoff(s["h0"])
    parts = []
    for b in range(len(s["first"]) - 1):
        x = {k: v[s["first"][b]:s["first"][b + 1]] for k, v in D.items()}
        if case["call"] == "gravity":
            parts.append({"acc": _gravity64(x["pos"], x["mass"], r_cut)})
            continue
        h, rho, f = _density64(x["pos"], x["mass"], x["h0"])
        acc, du, B, vs = _force64(x["pos"], x["vel"], x["mass"], x["u"], h, rho, f, bool(case.get("balsara", 0)))
        r = {"h": h, "rho": rho, "f": f, "acc": acc, "dudt": du}
        if B is not None:
            r["balsara"] = B
        if case["call"] == "step":
            r["vsig"] = vs
        parts.append(r)
    r = {k: torch.cat([p[k] for p in parts]) for k in parts[0]}
    if case["call"] != "step":
        return r
    dt = COURANT * float((r.pop("vsig")).reciprocal().mul(r["h"]).min())
    vel, u = D["vel"] + 0.5 * dt * r["acc"], D["u"] + 0.5 * dt * r["dudt"]
    pos = D["pos"] + dt * vel
    pos = pos - torch.floor(pos)
    vp, up = vel + 0.5 * dt * r["acc"], u + 0.5 * dt * r["dudt"]
    parts = []
    for b in range(len(s["first"]) - 1):
        k = slice(s["first"][b], s["first"][b + 1])
        h, rho, f = _density64(pos[k], D["mass"][k], r["h"][k])
        acc, du, _, _ = _force64(pos[k], vp[k], D["mass"][k], up[k], h, rho, f)
        parts.append({"h": h, "rho": rho, "f": f, "acc": acc, "dudt": du})
    n = {k: torch.cat([p[k] for p in parts]) for k in parts[0]}
    n.update(pos=pos, vel=vel + 0.5 * dt * n["acc"], u=u + 0.5 * dt * n["dudt"])
    return n
