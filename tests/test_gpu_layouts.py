"""The two layouts of the work items and the edges of the rules that choose
between them and between the list lengths, against the FP64 oracle.

A grid layout takes boxes of at least four top cells per side none of which
splits, and whose items of 16 particles span few enough cells; everything else
is a tree. The density lists have room for 80 to 448 entries by the number of
neighbours and the margin; a particle whose list is too short, or whose root
lies beyond it, is taken again with more room. Tolerances: parity.TOL32, which
holds for every FP32 result whatever the cells.
"""

import numpy as np
import pytest

import oracle
import workloads
from parity import TOL32, assert_within, errors

pytestmark = pytest.mark.gpu


def _lattice(side, seed):
    return workloads.lattice_box(side, [1508, 950, seed], jitter=0.3, u=1.0, vel_sigma=0.2)


def _clustered():
    return workloads.clustered(n_uniform=3000, n_spheres=3, per_sphere=900)


def _boxes():
    """Boxes of other lengths, one empty, one too small for a grid's sides."""
    parts, first, lens = [], [0], []
    for k, (side, L) in enumerate([(12, 2.5), (0, 1.0), (13, 0.3), (17, 40.0)]):
        lens.append(L)
        if side:
            d = _lattice(side, 20 + k)
            d["pos"] = d["pos"] * L
            d["h0"] = (d["h0"] * L).astype(np.float32)
            parts.append(d)
        first.append(first[-1] + (side**3 if side else 0))
    out = {k: np.concatenate([p[k] for p in parts], axis=0) for k in ("pos", "vel", "mass", "u", "h0")}
    out["box_first"] = np.asarray(first, dtype=np.int64)
    out["box_len"] = np.asarray(lens, dtype=np.float64)
    return out


# set, neighbours, factor on the guesses, masses from U(0.5, 1.5)
CASES = {
    "three_cells": (lambda: _lattice(11, 1), 48, 1.0, False),      # tree: G = 3
    "four_cells": (lambda: _lattice(12, 2), 48, 1.0, False),       # the smallest grid
    "items_too_long": (lambda: _lattice(8, 3), 16, 1.0, False),    # 16 particles span a column of four cells
    "few_neighbours": (lambda: _lattice(17, 4), 16, 1.0, False),
    "lists_128": (lambda: _lattice(15, 5), 60, 1.0, False),
    "lists_240": (lambda: _lattice(18, 6), 100, 1.0, False),
    "lists_448": (lambda: _lattice(21, 7), 200, 1.0, False),
    "guess_low": (lambda: _lattice(15, 8), 48, 0.85, False),       # every root beyond the first list
    "guess_high": (lambda: _lattice(20, 9), 48, 1.3, False),       # lists that do not fit
    "masses": (lambda: _lattice(15, 10), 40, 1.0, True),
    "boxes": (_boxes, 48, 1.0, False),
    "tree_few": (_clustered, 24, 1.0, False),
    "tree_34": (_clustered, 34, 1.0, False),
    "tree_low": (_clustered, 48, 0.85, False),
    "tree_high": (_clustered, 40, 1.3, False),
    "tree_masses": (_clustered, 48, 1.0, True),
    "tree_240": (_clustered, 80, 1.0, False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_layouts_match_oracle(gpu_lib, name):
    make, n_ngb, guess, mixed = CASES[name]
    d = make()
    n = d["pos"].shape[0]
    d["h0"] = (d["h0"] * guess * (n_ngb / 48.0) ** (1.0 / 3.0)).astype(np.float32)
    if mixed:
        d["mass"] = (d["mass"] * np.random.default_rng([1508, 951]).uniform(0.5, 1.5, n)).astype(np.float32)
    print("case", name, "N", n, flush=True)
    ctx = gpu_lib.Context(0, n_ngb=float(n_ngb))
    try:
        g = gpu_lib.run_workload(ctx, d)
    finally:
        ctx.close()
    r = oracle.run(d, n_ngb=float(n_ngb))
    e = errors(g, r)
    print(name, e, g["stats_density"], flush=True)
    assert_within(e, TOL32, name)
    # counts: equal up to pairs within FP32 rounding of r = h
    n_d, n_f = int(r["nngb"].sum()), int(r["npair"].sum())
    assert abs(g["stats_density"]["interactions_density"] - n_d) <= 1e-5 * n_d + 2
    assert abs(g["stats_force"]["interactions_force"] - n_f) <= 1e-5 * n_f + 2


@pytest.mark.parametrize("name", ["four_cells", "tree_few"])
@pytest.mark.parametrize("margin", [1.05, 1.26])
def test_listed_counts(gpu_lib, name, margin):
    """timing = 2 counts every particle inside each search radius, also where
    the lists stop short of it (wide margins) or the walk leaves out what the
    lists cannot reach (trees)."""
    import torch
    from scipy.spatial import cKDTree
    d = CASES[name][0]()
    ctx = gpu_lib.Context(0, timing=2, h_margin=margin)
    try:
        # guesses at the roots, so that nothing is rebuilt
        h0 = torch.from_numpy(oracle.run(d)["h"].astype(np.float32)).cuda()
        ctx.build_cells(torch.from_numpy(d["pos"]).cuda(), h0, d["box_first"], d["box_len"])
        st = ctx.density(torch.from_numpy(d["mass"]).cuda(), h0.clone())["stats"]
    finally:
        ctx.close()
    H = (np.float32(margin) * h0.cpu().numpy()).astype(np.float64)
    tree = cKDTree(np.mod(d["pos"], 1.0), boxsize=1.0)
    lo, hi = (int(tree.query_ball_point(np.mod(d["pos"], 1.0), H * s, return_length=True).sum())
              for s in (1.0 - 1e-5, 1.0 + 1e-5))
    print(name, margin, st, lo, hi, flush=True)
    assert st["rebuilds"] == 0 and lo <= st["listed_density"] <= hi


def test_leaf_of_many_particles(gpu_lib):
    """A leaf whose particles times items pass 2^31 (guesses far too wide for a
    clump of 200,000 keep it whole): gravity of a sample against the oracle,
    tolerance as in the gravity tests."""
    import torch
    from oracle import gravity as og
    from test_gpu_gravity import TOL, _window_free
    n, rc = 200_000, 0.01
    rng = np.random.default_rng([1508, 952])
    pos = rng.uniform(0.02, 0.12, (n, 3))
    print("leaf of", n, flush=True)
    ctx = gpu_lib.Context(0)
    try:
        ctx.build_cells(torch.from_numpy(pos).cuda(), torch.full((n,), 0.25, device="cuda"))
        assert ctx.build_info()["max_cell_particles"] == n
        acc = ctx.gravity_p2p(torch.ones(n, device="cuda"), 1.0, 1e-3, rc)[0].double().cpu().numpy()
    finally:
        ctx.close()
    rows = np.sort(rng.choice(n, 40, replace=False))
    o = og.p2p_rows(pos, np.ones(n), 1.0, 1e-3, rc, rows)["acc"]
    err = np.linalg.norm(acc[rows] - o, axis=1) / _window_free(pos, np.ones(n), 1.0, 1e-3, rc, rows=rows)
    print("errors", err.max(), flush=True)
    assert err.max() <= TOL
