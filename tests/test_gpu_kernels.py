"""GPU tests of single kernels at the sizes where they can go wrong, against the oracle."""
import numpy as np
import pytest

from workloads import polytrope_n1, uniform_random

from gpu_helpers import (gpu_density, gpu_forces, gpu_gravity, gpu_keys_order, gpu_neighbors, gpu_tree, make_ctx, parts,
                         to_np)

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------------------- key sort
# sizes around a thread's 8 keys, a merge output tile (2,048), a sort tile (4,096), and odd
# numbers of runs
SORT_SIZES = [1, 2, 7, 8, 9, 63, 65, 2047, 2048, 2049, 4095, 4096, 4097, 6143, 8192, 8193, 12289, 40961, 70001]


def _sort_set(n, family):
    ps = uniform_random(n, seed=900 + n % 97, h=1e-4)
    if family == "duplicates":   # 16 particles on each point: ties across tiles and runs
        k = np.random.default_rng(n).permutation(n) // 16
        for f in ("x", "y", "z", "vx", "vy", "vz"):
            setattr(ps, f, np.ascontiguousarray(getattr(ps, f)[k]))
    elif family == "one_point":
        for f in ("x", "y", "z"):
            setattr(ps, f, np.full(n, 0.25))
    elif family == "reversed":
        for f in ("x", "y", "z"):
            setattr(ps, f, np.linspace(1.0, 0.0, n))
    elif family == "top_cell":   # the last particles share the largest possible key
        for f in ("x", "y", "z"):
            getattr(ps, f)[n // 2:] = 1.5
    return ps


@pytest.mark.parametrize("family", ["random", "duplicates", "one_point", "reversed", "top_cell"])
def test_sort_sizes(orc, family):
    for n in SORT_SIZES:
        ps = _sort_set(n, family)
        ctx = make_ctx(n)
        k, o = gpu_keys_order(ctx, parts(ps))
        assert np.array_equal(k, orc.keys(ps.x, ps.y, ps.z)), n
        assert np.array_equal(o, orc.order(k)), n
        ctx.close()


@pytest.mark.parametrize("n", [9, 2049, 4097, 12289])
@pytest.mark.parametrize("family", ["random", "duplicates"])
def test_step_sort_ties_by_id(orc, n, family):
    """Steps sort from the previous key order; equal keys still come in the order of the IDs."""
    import torch
    import paper_2007_03097_amd as sph
    ps = _sort_set(n, family)
    ctx = make_ctx(n)
    pa = parts(ps, with_accel=True)
    keys = torch.zeros(n, dtype=torch.int64, device="cuda")
    order = torch.zeros(n, dtype=torch.int64, device="cuda")
    for flags in (sph.SPH_STEP_PRIMED, sph.SPH_STEP_RESUME, sph.SPH_STEP_RESUME):
        sph.sph_step(ctx.h, pa, 0.3, 1, flags)   # far enough to mix the order
        sph.sph_key_order(ctx.h, keys, order)
        k = to_np(keys).view(np.uint64)
        x, y, z = (to_np(pa[f]) for f in ("x", "y", "z"))
        assert np.array_equal(k, orc.keys(x, y, z))
        assert np.array_equal(to_np(order), orc.order(k))
        if family == "duplicates":
            assert np.unique(k).size < n
    ctx.close()


# ---------------------------------------------------------------------------- node moments
def _moment_set(case):
    if case == "shell":      # a dense core, an empty gap and a sparse shell: leaves at low levels
        ps = polytrope_n1(6000, seed=31)
        r = np.where(np.arange(ps.n) % 20 == 0, 1.0, 0.02)
        ps.x, ps.y, ps.z = ps.x * r, ps.y * r, ps.z * r
    elif case == "coincident":   # 150 particles on one point: a leaf over its capacity
        ps = polytrope_n1(3000, seed=32)
        for f in ("x", "y", "z"):
            getattr(ps, f)[500:650] = getattr(ps, f)[500]
    elif case == "flat":     # few cells per level
        ps = polytrope_n1(5000, seed=33)
        ps.y, ps.z = 0.003 * ps.y, 0.003 * ps.z
    else:
        ps = polytrope_n1(300, seed=34)
    ps.m = np.random.default_rng(35).uniform(0.5, 1.5, ps.n) / ps.n
    return ps


@pytest.mark.parametrize("leaf", [1, 7, 8, 33, 64])
@pytest.mark.parametrize("case", ["shell", "coincident", "flat", "small"])
def test_node_moments(orc, case, leaf):
    """Masses, centres, second moments and boxes of leaves and internal nodes, through the
    quadrupole field of the oracle's own walk on its own tree and moments: 99% of particles to
    1e-9 (the rest only where a borderline opening decision flips)."""
    ps = _moment_set(case)
    ctx = make_ctx(ps.n, theta=0.7, G=1.0, soft_eps=0.01, leaf_size=leaf, group_size=16)
    k, o = gpu_keys_order(ctx, parts(ps))
    g = np.stack(gpu_gravity(ctx, ps.n)[:3], axis=1)
    t = orc.octree(k[o], leaf)
    L = max(np.ptp(ps.x), np.ptp(ps.y), np.ptp(ps.z))
    cells = orc.octree(k[o], 64)
    gs, gc = [], []
    for s0, c0 in zip(cells["start"][cells["leaf"]], cells["count"][cells["leaf"]]):
        for j in range(0, int(c0), 16):
            gs.append(s0 + j)
            gc.append(min(16, int(c0) - j))
    ref = np.empty((ps.n, 3))
    ref[o] = np.stack(orc.tree_gravity(ps.x[o], ps.y[o], ps.z[o], ps.m[o], t, L, 0.7, 1.0, 0.01, np.array(gs),
                                       np.array(gc))[:3], axis=1)
    d = np.linalg.norm(g - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert np.quantile(d, 0.99) <= 1e-9 and d.max() <= 1e-2, (np.quantile(d, 0.99), d.max())


# ---------------------------------------------------------------------------- CSR lists
@pytest.mark.parametrize("n,h,group", [(700, (0.10, 0.2), 8),     # lists around and over a wave's 64 entries
                                       (64, 0.9, 64), (65, 0.9, 32), (129, 0.9, 64),   # exactly 64, 65, 129 entries
                                       (7603, (0.18, 0.26), 16)])  # unions over the 4,096 staged IDs
def test_csr_lists_of_any_length(orc, n, h, group):
    ps = uniform_random(n, seed=61, h=h)
    ctx = make_ctx(n, group_size=group, nbr_capacity=4096)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, n)
    ref = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    assert np.array_equal(off, ref[0]) and np.array_equal(idx, ref[1])
    longest = np.diff(off).max()
    assert longest == n if h == 0.9 else longest > 64


# ---------------------------------------------------------------------------- octree numbering
@pytest.mark.parametrize("n,leaf", [(255, 1), (256, 8), (257, 16), (1023, 13), (1024, 32), (1025, 64), (4097, 5),
                                    (262144, 24), (262145, 13), (264193, 32)])   # tiles of 256 and of 1,024 positions
def test_octree_at_tile_edges(orc, n, leaf):
    ps = uniform_random(n, seed=71)
    ps.x[: n // 3] *= 0.01     # deep and shallow parts
    ctx = make_ctx(n, leaf_size=leaf)
    k, o = gpu_keys_order(ctx, parts(ps))
    t, g = orc.octree(k[o], leaf), gpu_tree(ctx)
    for f in ("key", "level", "leaf", "start", "count"):
        a = np.lexsort((t["start"], t["level"]))
        assert np.array_equal(np.asarray(t[f])[a], g[f]), f   # breadth-first: by level, then position


@pytest.mark.parametrize("n", [1023, 1025, 2049])
def test_groups_at_tile_edges(orc, n):
    """Target groups that start and end around the group tiles: every particle in one group."""
    ps = uniform_random(n, seed=72, h=(0.02, 0.06))
    for group in (8, 64):
        ctx = make_ctx(n, group_size=group, nbr_capacity=512)
        gpu_keys_order(ctx, parts(ps))
        off, idx = gpu_neighbors(ctx, n)
        ref = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
        assert np.array_equal(off, ref[0]) and np.array_equal(idx, ref[1])


# ---------------------------------------------------------------------------- neighbour screen
@pytest.mark.parametrize("group", [8, 16, 32, 64])
@pytest.mark.parametrize("scale,shift", [(1.0, 0.0), (1e-25, 0.0), (1e-11, 0.0), (1e11, 0.0), (1e25, 0.0), (1.0, 1e7)])
def test_neighbors_at_any_scale(orc, scale, shift, group):
    """The screen's margin, its underflow term, the overflow rule (every pair exact) and offsets from a
    distant origin; h spread by 20, odd counts (part-filled groups and tiles)."""
    ps = uniform_random(1231, seed=83, h=(0.01, 0.2))
    for f in ("x", "y", "z"):
        setattr(ps, f, getattr(ps, f) * scale + shift)
    ps.h = ps.h * scale
    ctx = make_ctx(ps.n, group_size=group, nbr_capacity=1024)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, ps.n)
    ref = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    assert np.array_equal(off, ref[0]) and np.array_equal(idx, ref[1])


# ---------------------------------------------------------------------------- merge passes by rank
@pytest.mark.parametrize("family", ["random", "duplicates", "crowded"])
@pytest.mark.parametrize("n", [8193, 9217, 16385, 65536, 65537, 73729, 131073, 524288, 524289, 1048577])
def test_rank_merge(orc, n, family):
    """Passes of two, four and eight ways around the sizes where their number changes, last runs of one key
    and of a few, equal keys in every run, and keys that crowd in few places of the other runs (searched
    in memory, not in LDS)."""
    ps = _sort_set(n, family if family == "duplicates" else "random")
    if family == "crowded":
        for f in ("x", "y", "z"):
            a = getattr(ps, f)
            a[8192:] = 0.4 + 0.01 * a[8192:]
    ctx = make_ctx(n)
    k, o = gpu_keys_order(ctx, parts(ps))
    assert np.array_equal(k, orc.keys(ps.x, ps.y, ps.z)) and np.array_equal(o, orc.order(k))


# ---------------------------------------------------------------------------- pair sums
@pytest.mark.parametrize("group", [8, 64])
@pytest.mark.parametrize("scale", [1e-30, 1.0, 1e25])
def test_pair_sums_at_any_scale(orc, scale, group):
    """FP64 density and forces where r/h runs from 0 (coincident particles) over 1e-9 to the support's
    edge, lists from one entry to several batches, unions over several staged rounds.  Every operation
    of a term is within a few ulp, and u = 1 - r/2h loses no more than an ulp of 1 at the edge, where
    the term itself is that small beside the sum: 1e-12 of the sum of the terms' magnitudes."""
    ps = uniform_random(1503, seed=91, h=(0.01, 0.2))
    for f in ("x", "y", "z"):
        a = getattr(ps, f)
        a[1:40:2] = a[0:39:2]              # coincident pairs
        a[41:80:2] = a[40:79:2] + 1e-11    # pairs at about 1e-9 h
    for f in ("x", "y", "z", "h"):
        setattr(ps, f, getattr(ps, f) * scale)
    ctx = make_ctx(ps.n, group_size=group, nbr_capacity=2048)
    gpu_keys_order(ctx, parts(ps))
    got = gpu_density(ctx, ps.n)
    csr = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    ref = orc.density(ps.fields(), csr)
    for a, b in zip(got, ref):
        assert np.max(np.abs(a - b) / np.abs(b)) <= 1e-12
    ax, ay, az, du = gpu_forces(ctx, ps.n)
    r_ax, r_ay, r_az, r_du, Sa, Su = orc.forces(ps.fields(), ref[0], ref[1], ref[2], csr)
    assert np.all(np.sqrt((ax - r_ax) ** 2 + (ay - r_ay) ** 2 + (az - r_az) ** 2) <= 1e-12 * Sa)
    assert np.all(np.abs(du - r_du) <= 1e-12 * Su)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,group", [(4096, 8), (4097, 8), (8193, 16), (16384, 32), (16385, 32), (32769, 64)])
def test_pair_sums_of_every_workgroup_form(orc, n, group, prec):
    """Both sides of the set sizes at which the pair kernels take other workgroups and staging rounds;
    lists from a few to over 200 entries (h spread by four), unions of one to several rounds: 1e-12 (FP32C
    1e-6) of the sum of the terms' magnitudes."""
    h0 = (40.0 / (n * 32.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
    ps = uniform_random(n, seed=96, h=(0.5 * h0, 2.0 * h0))
    tol = (1e-12, 1e-6)[prec]
    ctx = make_ctx(n, group_size=group, nbr_capacity=2048, precision=prec)
    gpu_keys_order(ctx, parts(ps))
    rho, P, c, hn = gpu_density(ctx, n)
    csr = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    ref = orc.density(ps.fields(), csr)
    for a, b in zip((rho, P, c, hn), ref):
        assert np.max(np.abs(a - b) / np.abs(b)) <= tol
    ax, ay, az, du = gpu_forces(ctx, n)
    r_ax, r_ay, r_az, r_du, Sa, Su = orc.forces(ps.fields(), rho, P, c, csr)
    assert np.all(np.sqrt((ax - r_ax) ** 2 + (ay - r_ay) ** 2 + (az - r_az) ** 2) <= tol * Sa)
    assert np.all(np.abs(du - r_du) <= tol * Su)


# ---------------------------------------------------------------------------- node-node gravity
@pytest.mark.parametrize("eps", [0.0, 0.02])
@pytest.mark.parametrize("leaf", [1, 2, 3, 31, 32, 33, 63, 64])
def test_fmm_leaf_populations(orc, leaf, eps):
    """Leaves of one to 64 targets (two a lane, odd counts) and, past 64, several passes over a leaf:
    within 1e-12 of each particle's absolute-sum scale."""
    import paper_2007_03097_amd as sph
    ps = uniform_random(1999, seed=92)
    if eps > 0.0:
        for f in ("x", "y", "z"):
            getattr(ps, f)[:131] = getattr(ps, f)[0]    # one leaf of 131: 64 + 64 + 3
    ctx = make_ctx(ps.n, theta=0.6, G=1.0, soft_eps=eps, leaf_size=leaf, gravity_scheme=sph.SPH_GRAVITY_FMM)
    k, o = gpu_keys_order(ctx, parts(ps))
    gx, gy, gz, phi = gpu_gravity(ctx, ps.n)
    box = orc.bbox(ps.x, ps.y, ps.z)
    r = orc.fmm_gravity(ps.x[o], ps.y[o], ps.z[o], ps.m[o], orc.octree(k[o], leaf), box, orc.scale(box, 21), 0.6, 1.0, eps)
    d = np.sqrt((gx[o] - r["gx"]) ** 2 + (gy[o] - r["gy"]) ** 2 + (gz[o] - r["gz"]) ** 2)
    assert np.max(d / r["sg"]) <= 1e-12 and np.max(np.abs(phi[o] - r["phi"]) / r["sp"]) <= 1e-12


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,group", [(1, 8), (501, 16), (3001, 64), (33001, 32), (70001, 16)])
def test_gravity_wavefronts_a_group(orc, n, group, prec):
    """One, two and four wavefronts a group (by the number of groups), odd populations, and a grid of one
    wavefront per compute unit that loops over the groups: the direct sum's field at theta = 0 for the
    small sets, and the same bits from both grids."""
    ps = uniform_random(n, seed=93)
    out = []
    for waves in (0, 1):
        ctx = make_ctx(n, theta=0.0 if n < 4000 else 0.6, G=1.0, soft_eps=0.01, group_size=group, leaf_size=16,
                       precision=prec, waves_per_cu=waves)
        gpu_keys_order(ctx, parts(ps))
        out.append(np.stack(gpu_gravity(ctx, n)))
    assert np.array_equal(out[0], out[1])
    if n < 4000:
        gx, gy, gz, phi, sg = orc.gravity_direct(ps.x, ps.y, ps.z, ps.m, 1.0, 0.01, scale=True)
        d = np.sqrt(((out[0][:3] - np.stack([gx, gy, gz])) ** 2).sum(0))
        assert np.all(d <= (1e-12, 1e-6)[prec] * sg + 1e-300)


@pytest.mark.parametrize("prec", [0, 1])
def test_fmm_heavy_leaf(orc, prec):
    """Few particles in a cell far larger than its neighbours' (heavy leaves), and a grid of one wavefront
    per compute unit that loops over heavy and other leaves."""
    import paper_2007_03097_amd as sph
    ps = uniform_random(90001, seed=94)
    ps.x[7:] *= 0.11
    ps.y[7:] *= 0.11
    ps.z[7:] *= 0.11      # seven particles of the unit box, the others near a corner of it
    out = []
    for waves in (0, 1):
        ctx = make_ctx(ps.n, theta=0.6, G=1.0, soft_eps=0.01, leaf_size=16, precision=prec, waves_per_cu=waves,
                       gravity_scheme=sph.SPH_GRAVITY_FMM)
        k, o = gpu_keys_order(ctx, parts(ps))
        out.append(np.stack(gpu_gravity(ctx, ps.n)))
    assert np.array_equal(out[0], out[1])
    box = orc.bbox(ps.x, ps.y, ps.z)
    r = orc.fmm_gravity(ps.x[o], ps.y[o], ps.z[o], ps.m[o], orc.octree(k[o], 16), box, orc.scale(box, 21), 0.6, 1.0, 0.01)
    d = np.sqrt(((out[0][:3][:, o] - np.stack([r["gx"], r["gy"], r["gz"]])) ** 2).sum(0))
    assert np.all(d <= (1e-12, 1e-6)[prec] * r["sg"])


@pytest.mark.parametrize("waves", [0, 1])
@pytest.mark.parametrize("n,group", [(4103, 8), (4105, 8), (12807, 8), (12809, 8), (32769, 64), (32833, 64), (3, 64)])
def test_neighbors_wavefronts_a_group(orc, n, group, waves):
    """Both sides of the numbers of groups at which one, two or four wavefronts share a group's matching;
    tiles that only some of them have; and a grid that loops over the groups."""
    ps = uniform_random(n, seed=95, h=(0.5 * n ** (-1.0 / 3), 2.0 * n ** (-1.0 / 3)))
    ctx = make_ctx(n, group_size=group, nbr_capacity=1024, waves_per_cu=waves)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, n)
    ref = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    assert np.array_equal(off, ref[0]) and np.array_equal(idx, ref[1])
