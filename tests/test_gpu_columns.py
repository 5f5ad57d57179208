"""Grid layouts with few particles along a column, against the FP64 oracle.

A grid layout cuts every column of top cells into items of at most 16
consecutive particles. Where the columns are sparse (few neighbours asked for, or
a body in an otherwise empty box) 16 of them lie over much of the box, which the
frames of the items have to cover without tearing a pair apart. Tolerances:
parity.TOL32, and those of the near-field gravity tests.
"""

import time

import numpy as np
import pytest

import oracle
import workloads
from oracle import gravity as og
from parity import TOL32, assert_within, errors
from test_gpu_gravity import TOL, _window_free

pytestmark = pytest.mark.gpu


def _body(n, inside, seed):
    """Points of an n^3 jittered lattice in the unit box for which inside(x) holds
    (x in lattice spacings), the rest of the box empty."""
    rng = np.random.default_rng([1508, 960, seed])
    x = np.stack(np.meshgrid(*[np.arange(n) + 0.5] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    p = (x + rng.uniform(-0.2, 0.2, x.shape))[inside(x)]
    m = p.shape[0]
    return {"pos": np.mod(p / n, 1.0), "vel": rng.normal(0.0, 0.2, (m, 3)).astype(np.float32),
            "mass": np.full(m, 1.0 / n**3, np.float32), "u": np.ones(m, np.float32),
            "h0": np.full(m, np.cbrt(3.0 * 48.0 / (4.0 * np.pi)) / n, np.float32),
            "box_first": np.array([0, m], np.int64), "box_len": np.array([1.0])}


def _cylinder(n, radius):
    return _body(n, lambda x: ((x[:, :2] - n / 2) ** 2).sum(1) < radius * radius, n)


# set, neighbours, h_margin
SETS = {
    "lattice_16": (lambda: workloads.lattice_box(16, [1508, 960, 0], jitter=0.2, vel_sigma=0.2), 12.0, 1.1),
    "lattice_13": (lambda: workloads.lattice_box(13, [1508, 960, 2], jitter=0.3, vel_sigma=0.2), 12.0, 1.05),
    "cylinder_24": (lambda: _cylinder(24, 7), 48.0, 1.26),
}


def _set(name):
    """The set with its smoothing lengths for guesses (so no cells are rebuilt),
    and the oracle's results."""
    make, n_ngb, margin = SETS[name]
    d = make()
    d["h0"] = (d["h0"] * np.cbrt(n_ngb / 48.0)).astype(np.float32)
    r = oracle.run(d, n_ngb=n_ngb)
    d["h0"] = r["h"].astype(np.float32)
    return d, r, n_ngb, margin


def _columns(d, margin):
    """(G, the particles of each column of top cells in order of z), by the rule
    of the cell build for one box of side 1."""
    H = float((np.float32(margin) * d["h0"]).max())
    G = int(np.floor(1.0 / H))
    xy = np.minimum(np.floor(d["pos"][:, :2] * G).astype(int), G - 1)
    col = xy[:, 0] * G + xy[:, 1]
    order = np.lexsort((d["pos"][:, 2], col))
    return G, np.split(order, np.flatnonzero(np.diff(col[order])) + 1)


def _longest_run(d, margin):
    """Largest extent in z of 16 consecutive particles of a column (in runs from its first)."""
    _, cols = _columns(d, margin)
    z = d["pos"][:, 2]
    return max(z[c[min(i + 15, len(c) - 1)]] - z[c[i]] for c in cols for i in range(0, len(c), 16))


@pytest.mark.parametrize("name", list(SETS))
def test_runs_longer_than_half_the_box(gpu_lib, name):
    """Density, force and gravity where 16 particles of a column lie over more
    than half the box, and again after a drift that keeps the cells."""
    import torch
    d, r, n_ngb, margin = _set(name)
    assert _longest_run(d, margin) > 0.5
    print("columns", name, "N", len(d["h0"]), "G", _columns(d, margin)[0], "run", _longest_run(d, margin), flush=True)
    rc = 0.95 * float(d["h0"].min())
    t = {k: torch.from_numpy(d[k]).cuda() for k in ("pos", "vel", "mass", "u", "h0")}
    # a drift of a third of the margin's budget: delta is sqrt(3) times the largest component
    budget = (1.0 - 1.0 / margin) * margin * float(d["h0"].min())
    dt = 0.5 * budget / 3.0 / np.sqrt(3.0) / float(np.abs(d["vel"]).max())
    ctx = gpu_lib.Context(0, n_ngb=n_ngb, h_margin=margin)
    try:
        ctx.build_cells(t["pos"], t["h0"], d["box_first"], d["box_len"])
        for step in range(2):
            if step:
                ctx.drift(dt, t["vel"], t["pos"])
                d = dict(d, pos=t["pos"].cpu().numpy())
                r = oracle.run(d, n_ngb=n_ngb)
            acc = ctx.gravity_p2p(t["mass"], 1.0, 0.0, rc)[0].double().cpu().numpy()
            nw = torch.empty_like(t["h0"])
            g = ctx.density(t["mass"], t["h0"].clone(), nw=nw)
            assert g["stats"]["rebuilds"] == 0 and ctx.timings()["builds"] == 1
            g.update(ctx.force(t["vel"], t["u"]))
            out = {k: g[k].double().cpu().numpy() for k in ("h", "rho", "f", "nw", "acc", "dudt")}
            e = errors(out, r)
            o = og.p2p(d["pos"], d["mass"], 1.0, 0.0, rc)
            W = _window_free(d["pos"], d["mass"], 1.0, 0.0, rc)
            eg = float(np.max(np.linalg.norm(acc - o["acc"], axis=1) / np.where(W > 0, W, 1.0)))
            print(name, "step", step, e, "gravity", eg, flush=True)
            assert_within(e, TOL32, name)
            assert eg <= TOL
    finally:
        ctx.close()


def test_separations_in_sparse_columns(gpu_lib):
    """The pull between the two particles of close pairs, in columns of 16 cells of
    width w with 40 particles each, is as exact as offsets from cell centres make
    it: an item spans at most two cells, so coordinates of at most w from its centre
    are rounded twice (32-bit fraction to FP32, times the unit), each by at most
    2^-25 w (w a power of two), and the separation along z is off by at most 2^-23 w,
    along x and y by half of that. The pull m / r^2 is then off by 2 |dr| / r of
    itself (1e-4 of that bound for the FP32 arithmetic of the pull)."""
    import torch
    G, margin = 16, 1.26
    w = 1.0 / G
    rng = np.random.default_rng([1508, 961])
    n, r = 20 * G * G, 2e-4 * w
    a = rng.uniform(0.0, 1.0, (n, 3))
    e = rng.normal(0.0, 1.0, (n, 3))
    pos = np.mod(np.concatenate([a, a + r * e / np.linalg.norm(e, axis=1)[:, None]]), 1.0)
    d = {"pos": pos, "h0": np.full(2 * n, 0.06249 / margin, np.float32)}
    assert _columns(d, margin)[0] == G and 8 * w < _longest_run(d, margin) < 13 * w
    mass = np.full(2 * n, 1.0, np.float32)
    rc = 0.9 * float(d["h0"][0])
    print("close pairs", n, "run", _longest_run(d, margin) / w, flush=True)
    ctx = gpu_lib.Context(0, h_margin=margin)
    try:
        ctx.build_cells(torch.from_numpy(pos).cuda(), torch.from_numpy(d["h0"]).cuda())
        acc = ctx.gravity_p2p(torch.from_numpy(mass).cuda(), 1.0, 0.0, rc)[0].double().cpu().numpy()
    finally:
        ctx.close()
    o = og.p2p(pos, mass, 1.0, 0.0, rc)["acc"]
    off = np.linalg.norm(acc - o, axis=1) / np.linalg.norm(o, axis=1) * r
    print("separations off by", off.max() / 2 / w, "w, rms", np.sqrt((off**2).mean()) / 2 / w, flush=True)
    assert off.max() <= 2.0 * np.sqrt(1.5) * 2.0**-23 * w * 1.0001


def test_separations_on_a_fine_grid(gpu_lib):
    """The pull between the two particles of close pairs on 256 cells a side (2^22
    particles, 16 pairs in a clump 2e-3 of a cell wide in two cells of every column,
    at any place of the cell), from which the error of each separation follows: the
    pull r / r^3 changes by (e - 3 (e . r) r / r^2) / r^3 for an error e. Offsets from
    cell centres are rounded by at most 2^-26 of the width w in half of the cell, 2^-27
    in a quarter and so on, 0.4365 x 2^-26 w rms, so separations are off by 1.069 x
    2^-26 w rms (six of those); 5% for the sample's own spread."""
    import torch
    G, margin = 256, 1.26
    w = 1.0 / G
    rng = np.random.default_rng([1508, 962])
    xy = np.repeat(np.stack(np.meshgrid(np.arange(G), np.arange(G), indexing="ij"), axis=-1).reshape(-1, 2), 2, axis=0)
    z = np.tile([60, 190], G * G)
    centre = (np.concatenate([xy, z[:, None]], axis=1) + rng.uniform(0.01, 0.99, (2 * G * G, 3))) * w
    a = centre[:, None] + rng.uniform(-1e-3, 1e-3, (2 * G * G, 16, 3)) * w
    e = rng.normal(0.0, 1.0, a.shape)
    pos = np.concatenate([a, a + 1e-5 * w * e / np.linalg.norm(e, axis=2)[..., None]], axis=1).reshape(-1, 3)
    n = pos.shape[0]
    h0 = np.full(n, 0.9999 * w / margin, np.float32)
    print("clumps", 2 * G * G, "particles", n, flush=True)
    ctx = gpu_lib.Context(0, h_margin=margin)
    try:
        ctx.build_cells(torch.from_numpy(pos).cuda(), torch.from_numpy(h0).cuda())
        assert ctx.build_info()["n_cells"] >= 2 * G * G
        acc = ctx.gravity_p2p(torch.ones(n, device="cuda"), 1.0, 0.0, 0.01 * w)[0].double().cpu().numpy()
    finally:
        ctx.close()
    off = []
    for k in rng.choice(2 * G * G, 400, replace=False):
        p = pos[32 * k:32 * k + 32]
        d = p[None] - p[:, None]
        r = np.linalg.norm(d, axis=2) + 1e9 * np.eye(32)
        pull = np.where(r < 0.01 * w, (1.0 - (r / (0.01 * w)) ** 2) ** 2, 0.0)[..., None] * d / r[..., None] ** 3
        da = acc[32 * k:32 * k + 32] - pull.sum(1)
        to = d[np.arange(32), np.arange(32) ^ 16]  # to the other particle of the pair
        r = np.linalg.norm(to, axis=1)[:, None]
        along = (da * to).sum(1)[:, None] * to / r**2
        off.append((da - 1.5 * along) * r**3)
    rms = float(np.sqrt((np.concatenate(off) ** 2).sum(1).mean()))
    print("separations off by", rms / w, "w rms", flush=True)
    assert rms <= 1.05 * 1.069 * 2.0**-26 * w


def test_empty_stretches_do_not_hold_up_a_build(gpu_lib):
    """A build whose grid is mostly empty (a cylinder of 455,000 particles, 47 cells a
    side) takes no more than five times that of a full box of as many particles (0.23
    ms; one thread over the longest empty stretch took 5 ms): the best of eight."""
    import torch
    best = []
    for d in (_cylinder(112, 36), workloads.lattice_box(77, [1508, 963], jitter=0.2)):
        t = {k: torch.from_numpy(d[k]).cuda() for k in ("pos", "h0")}
        ctx = gpu_lib.Context(0, h_margin=1.05)
        try:
            times = []
            for _ in range(8):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                ctx.build_cells(t["pos"], t["h0"])
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
        finally:
            ctx.close()
        best.append(min(times))
    print("builds, s:", best, flush=True)
    assert best[0] <= 5.0 * best[1]
