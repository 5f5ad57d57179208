"""Builds within sph_params.workspace_limit: what the tree layout alone has room for
is accepted, whatever the grid layout's tables would have taken."""

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

MARGIN = 1.05


def _sparse_with_a_clump(n=20000, cells=40):
    """Sparse points on `cells` cells a side, whose table of fine cells takes 50
    bytes per particle, and 200 points in one cell, which splits it: a tree."""
    rng = np.random.default_rng([1508, 980])
    pos = rng.uniform(0.0, 1.0, (n, 3))
    pos[:200] = (rng.integers(5, cells - 5, 3) + rng.uniform(0.1, 0.9, (200, 3))) / cells
    return pos, np.full(n, 0.9999 / cells / MARGIN, np.float32)


def _build(gpu_lib, limit, pos, h0, first=None, ctx=None):
    """The context with its cells, or None if memory runs out."""
    import torch
    new = ctx or gpu_lib.Context(0, h_margin=MARGIN, workspace_limit=limit)
    try:
        new.build_cells(torch.from_numpy(pos).cuda(), torch.from_numpy(h0).cuda(), first,
                        None if first is None else [1.0] * (len(first) - 1))
        return new
    except gpu_lib.SphError as e:
        assert e.code == gpu_lib.SPH_E_NOMEM
        if ctx is None:
            new.close()
        return None


def test_a_tree_fits_without_the_grids_tables(gpu_lib):
    """The smallest limit for the set and a box of 27 wide particles, which rules a
    grid out from the start, is enough for the set alone, which tries the grid
    first; also in a context that holds the tables of an earlier grid."""
    import torch
    pos, h0 = _sparse_with_a_clump()
    small = workloads.lattice_box(3, [1508, 981], jitter=0.1)["pos"]
    both, hb = np.concatenate([pos, small]), np.concatenate([h0, np.full(27, 0.3, np.float32)])
    first = [0, len(pos), len(pos) + 27]
    lo, hi = 0, 64 << 20
    while hi - lo > 8192:
        mid = (lo + hi) // 2
        ctx = _build(gpu_lib, mid, both, hb, first)
        lo, hi = (lo, mid) if ctx else (mid, hi)
        if ctx:
            ctx.close()
    print("tree alone: %d bytes" % hi, flush=True)
    mass = torch.ones(len(pos), device="cuda")
    acc = []
    grid = workloads.lattice_box(20, [1508, 982], jitter=0.1)
    for limit, before in ((0, False), (hi + mass.numel() * 32, False), (hi + mass.numel() * 32, True)):
        # (32 bytes per particle more: the gravity's own buffer and the earlier grid's positions)
        build_limit = limit if before or not limit else hi
        ctx = _build(gpu_lib, build_limit, pos, h0)
        assert ctx, limit
        ctx.close()
        ctx = gpu_lib.Context(0, h_margin=MARGIN, workspace_limit=limit)
        try:
            if before:
                assert _build(gpu_lib, limit, grid["pos"], grid["h0"], ctx=ctx)
            assert _build(gpu_lib, limit, pos, h0, ctx=ctx), limit
            acc.append(ctx.gravity_p2p(mass, 1.0, 1e-3, 0.9 * float(h0[0]))[0].cpu().numpy())
        finally:
            ctx.close()
    assert np.array_equal(acc[0], acc[1]) and np.array_equal(acc[0], acc[2])


def test_a_rebuild_without_room_leaves_no_cells(gpu_lib):
    """Limits that have room for the first cells but not for those of a rebuild (the
    guesses are much too small, and the lists of the wider cells longer): every call
    on the half-made cells is refused, and the context takes new ones."""
    import torch
    d = workloads.clustered(n_uniform=20000, n_spheres=4, per_sphere=2000)
    t = {k: torch.from_numpy(d[k]).cuda() for k in ("pos", "vel", "mass", "u", "h0")}
    n = t["h0"].numel()
    low = (0.7 * t["h0"]).contiguous()
    small = workloads.lattice_box(10, [1508, 983], jitter=0.1)
    refused = 0
    for limit in np.geomspace(5e6, 30e6, 80).astype(int).tolist():
        ctx = gpu_lib.Context(0, workspace_limit=limit)
        try:
            ctx.build_cells(t["pos"], low)
            try:
                ctx.density(t["mass"], low.clone())
                continue
            except gpu_lib.SphError as e:
                assert e.code == gpu_lib.SPH_E_NOMEM
            calls = (lambda: ctx.density(t["mass"], low.clone()), lambda: ctx.force(t["vel"], t["u"]),
                     lambda: ctx.pass_(t["mass"], low.clone(), t["vel"], t["u"]),
                     lambda: ctx.drift(1e-9, t["vel"], t["pos"]), lambda: ctx.gravity_p2p(t["mass"], 1.0, 0.0, 1e-4),
                     lambda: ctx.density_f64(t["mass"].double(), low.double()))
            codes = []
            for call in calls:
                try:
                    call()
                    codes.append(0)
                except gpu_lib.SphError as e:
                    codes.append(e.code)
            if codes[0] == gpu_lib.SPH_E_STATE:  # the cells are gone (not only a buffer of the density)
                refused += 1
                assert set(codes) == {gpu_lib.SPH_E_STATE}, codes
            ctx.build_cells(torch.from_numpy(small["pos"]).cuda(), torch.from_numpy(small["h0"]).cuda())
            ctx.density(torch.from_numpy(small["mass"]).cuda(), torch.from_numpy(small["h0"]).cuda())
        except gpu_lib.SphError as e:
            assert e.code == gpu_lib.SPH_E_NOMEM  # no room for the first cells
        finally:
            ctx.close()
    print("rebuilds refused:", refused, "N", n, flush=True)
    assert refused > 0
