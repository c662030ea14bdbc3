"""GPU tests of what the kernels' forms depend on besides a set's size: the units of the input, the rounding of
the FP64 terms, group and set populations, uneven sets and caps on the grid."""
import numpy as np
import pytest

from workloads import uniform_random

from gpu_helpers import gpu_density, gpu_keys_order, make_ctx, parts

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------------------- rounding of the density
def _density_exact(ps, csr):
    """The density sum in 80-bit floating point (5e-20 a term)."""
    off, idx = csr
    L = np.longdouble
    a = np.repeat(np.arange(ps.n), np.diff(off))
    r2 = sum((getattr(ps, f).astype(L)[a] - getattr(ps, f).astype(L)[idx]) ** 2 for f in ("x", "y", "z"))
    h = ps.h.astype(L)
    H = (h[a] + h[idx]) / 2
    q = np.sqrt(r2) / H
    w = np.where(q < 1, 1 - L(1.5) * q * q + L(0.75) * q * q * q, (2 - q) ** 3 / 4)
    t = ps.m.astype(L)[idx] * w / (H * H * H)
    return np.add.reduceat(t, off[:-1]) / L("3.14159265358979323846264338327950288")


@pytest.mark.parametrize("spread", [True, False])
def test_density_rounding(orc, spread):
    """RMS rounding error of FP64 densities over h spread by two, and over 24 sets of one h each.  With terms from
    a correctly rounded square root and reciprocal of their own it is 1.57e-16 to 1.61e-16 and 1.57e-16 to 1.70e-16
    (an emulation over several seeds): no more than 1.65e-16."""
    err = []
    for k in range(2 if spread else 24):
        n = 6000 if spread else 1500
        h0 = (80.0 / (n * 32.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
        ps = uniform_random(n, seed=300 + k, h=(0.5 * h0, h0) if spread else 0.8 * h0)
        ps.m = np.random.default_rng(400 + k).uniform(0.5, 1.5, n) / n
        s = np.exp(np.random.default_rng(500 + k).uniform(0.0, 3.0))
        for f in ("x", "y", "z", "h"):
            setattr(ps, f, getattr(ps, f) * s)
        ctx = make_ctx(n, nbr_capacity=512)
        gpu_keys_order(ctx, parts(ps))
        ref = _density_exact(ps, orc.neighbors(ps.x, ps.y, ps.z, ps.h))
        err.append((gpu_density(ctx, n)[0] - ref) / ref)
        ctx.close()
    rms = float(np.sqrt(np.mean(np.concatenate(err) ** 2)))
    assert rms <= 1.65e-16, rms


# ---------------------------------------------------------------------------- units
@pytest.mark.parametrize("group", [8, 32])
@pytest.mark.parametrize("scale", [1e-95, 1e-75, 1e-66, 1e76, 1e90, 1e95])
def test_density_in_any_unit(orc, scale, group):
    """FP64 density where r^2 and h^2 are representable but their product is not, coincident pairs among
    them: 1e-12 of the sum, every term being positive and within a few ulp."""
    ps = uniform_random(1200, seed=97, h=(0.05, 0.2))
    for f in ("x", "y", "z"):
        a = getattr(ps, f)
        a[1:40:2] = a[0:39:2]
    for f in ("x", "y", "z", "h"):
        setattr(ps, f, getattr(ps, f) * scale)
    ctx = make_ctx(ps.n, group_size=group, nbr_capacity=1024)
    gpu_keys_order(ctx, parts(ps))
    rho, P, c, hn = gpu_density(ctx, ps.n)
    ref = orc.density(ps.fields(), orc.neighbors(ps.x, ps.y, ps.z, ps.h))
    for a, b in zip((rho, P, c, hn), ref):
        assert np.all(np.abs(a / b - 1.0) <= 1e-12)


@pytest.mark.parametrize("group", [8, 64])
@pytest.mark.parametrize("scale", [1e-158, 1e-140, 1e-119, 1e-14, 3e18, 1e121, 1e140, 1e154])
def test_neighbors_in_any_unit(orc, scale, group):
    """The list kernel's screen in units of the group's reach: coordinates far outside the FP32 range, both sides of
    the reaches (2^-400, 2^400) past which every pair takes the FP64 predicate, and units in which that
    predicate's squares vanish or overflow."""
    from gpu_helpers import gpu_neighbors
    ps = uniform_random(1231, seed=98, h=(0.01, 0.2))
    for f in ("x", "y", "z", "h"):
        setattr(ps, f, getattr(ps, f) * scale)
    ctx = make_ctx(ps.n, group_size=group, nbr_capacity=1024)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, ps.n)
    ref = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    assert np.array_equal(off, ref[0]) and np.array_equal(idx, ref[1])


# ---------------------------------------------------------------------------- quadrupole gravity
@pytest.mark.parametrize("group", [8, 32])
@pytest.mark.parametrize("per", [1, 2, 3, 5, 9, 15, 16, 17, 31])
def test_gravity_of_small_groups(orc, per, group):
    """Groups of one to 31 targets, whose partial sums (up to 256 a target, by two or four wavefronts) are added
    in one or two rounds: each set's direct sum at theta = 0, with and without the potential's self term."""
    from gpu_helpers import gpu_gravity
    ps = uniform_random(40 * per, seed=99)
    ps.seg_offsets = np.arange(41, dtype=np.int64) * per
    for eps in (0.05, 0.0):
        ctx = make_ctx(ps.n, 40, theta=0.0, G=1.0, soft_eps=eps, group_size=group)
        gpu_keys_order(ctx, parts(ps))
        got = np.stack(gpu_gravity(ctx, ps.n))
        for i, j in zip(ps.seg_offsets[:-1], ps.seg_offsets[1:]):
            gx, gy, gz, phi, sg = orc.gravity_direct(ps.x[i:j], ps.y[i:j], ps.z[i:j], ps.m[i:j], 1.0, eps, scale=True)
            d = np.sqrt(((got[:3, i:j] - np.stack([gx, gy, gz])) ** 2).sum(0))
            assert np.all(d <= 1e-12 * sg + 1e-300)
            assert np.all(np.abs(got[3, i:j] - phi) <= 1e-12 * (np.abs(phi) + (ps.m[i:j] / eps if eps else 0.0)))
        ctx.close()


# ---------------------------------------------------------------------------- ensembles of small sets
@pytest.mark.parametrize("sets,per,group", [(400, 1, 64), (512, 2, 8), (512, 2, 64), (90, 64, 32), (90, 65, 32)])
def test_ensembles_of_small_sets(orc, sets, per, group):
    """Many more groups than n over the group size (each set ends with one of its own), and both sides of the
    sets of one tile that one wavefront a group serves: lists, density and gravity of every set."""
    from gpu_helpers import gpu_gravity, gpu_neighbors
    n = sets * per
    ps = uniform_random(n, seed=101, h=(0.1, 0.3))
    ps.seg_offsets = np.arange(sets + 1, dtype=np.int64) * per
    ctx = make_ctx(n, sets, theta=0.0, G=1.0, soft_eps=0.05, group_size=group)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, n)
    rho = gpu_density(ctx, n)[0]
    got = np.stack(gpu_gravity(ctx, n))
    for i in range(0, n, per):
        f = {k: getattr(ps, k)[i:i + per] for k in ("x", "y", "z", "vx", "vy", "vz", "m", "h", "u")}
        csr = orc.neighbors(f["x"], f["y"], f["z"], f["h"])
        assert np.array_equal(np.diff(off[i:i + per + 1]), np.diff(csr[0]))
        assert np.array_equal(idx[off[i]:off[i + per]] - i, csr[1])
        assert np.all(np.abs(rho[i:i + per] / orc.density(f, csr)[0] - 1.0) <= 1e-12)
        gx, gy, gz, _, sg = orc.gravity_direct(f["x"], f["y"], f["z"], f["m"], 1.0, 0.05, scale=True)
        d = np.sqrt(((got[:3, i:i + per] - np.stack([gx, gy, gz])) ** 2).sum(0))
        assert np.all(d <= 1e-12 * sg + 1e-300)


# ---------------------------------------------------------------------------- node-node gravity
@pytest.mark.parametrize("theta", [0.69, 0.7])
@pytest.mark.parametrize("leaf", [16, 17, 32, 33])
def test_fmm_of_heavy_leaves(orc, leaf, theta):
    """Both sides of the leaf sizes and the angle at which a lane takes one target or two, in a set of few
    leaves, most of them heavy (a workgroup each), on the full grid and on one that loops over the leaves."""
    import paper_2007_03097_amd as sph
    from gpu_helpers import gpu_gravity
    ps = uniform_random(7001, seed=102)
    out = []
    for waves in (0, 1):
        ctx = make_ctx(ps.n, theta=theta, G=1.0, soft_eps=0.01, leaf_size=leaf, waves_per_cu=waves,
                       gravity_scheme=sph.SPH_GRAVITY_FMM)
        k, o = gpu_keys_order(ctx, parts(ps))
        out.append(np.stack(gpu_gravity(ctx, ps.n)))
        ctx.close()
    assert np.array_equal(out[0], out[1])
    box = orc.bbox(ps.x, ps.y, ps.z)
    r = orc.fmm_gravity(ps.x[o], ps.y[o], ps.z[o], ps.m[o], orc.octree(k[o], leaf), box, orc.scale(box, 21), theta, 1.0, 0.01)
    d = np.sqrt(((out[0][:3, o] - np.stack([r["gx"], r["gy"], r["gz"]])) ** 2).sum(0))
    assert np.all(d <= 1e-12 * r["sg"]) and np.all(np.abs(out[0][3, o] - r["phi"]) <= 1e-12 * r["sp"])


# ---------------------------------------------------------------------------- node moments of uneven sets
@pytest.mark.parametrize("case", ["cluster", "clusters", "point"])
def test_moments_of_uneven_sets(orc, case):
    """Sets of more than 2^18 particles, whose subtrees are handed out by their number of particles: half of them in
    one cell of the first levels, in cells of several depths, and on one point (a chain of nodes that
    each hold them all).  Masses, centres and second moments through the quadrupole field of the oracle's walk on its
    own tree: 99% of particles to 1e-9, the rest only where a borderline opening decision flips."""
    from gpu_helpers import gpu_gravity
    n = 270_001
    ps = uniform_random(n, seed=103)
    rng = np.random.default_rng(104)
    ps.m = rng.uniform(0.5, 1.5, n) / n
    if case == "cluster":
        for f in ("x", "y", "z"):
            getattr(ps, f)[: n // 2] = 0.5 + 1e-3 * getattr(ps, f)[: n // 2]
    elif case == "clusters":
        for k, w in enumerate((1e-1, 1e-2, 1e-3, 1e-4)):
            c = rng.uniform(0.1, 0.9, 3)
            for f, o in zip(("x", "y", "z"), c):
                a = getattr(ps, f)[k * 50_000:(k + 1) * 50_000]
                a[:] = o + w * (a - 0.5)
    else:
        for f in ("x", "y", "z"):
            getattr(ps, f)[:3000] = 0.3
    ctx = make_ctx(n, theta=0.8, G=1.0, soft_eps=0.01, leaf_size=32, group_size=64)
    k, o = gpu_keys_order(ctx, parts(ps))
    g = np.stack(gpu_gravity(ctx, n)[:3], axis=1)
    t, cells = orc.octree(k[o], 32), orc.octree(k[o], 256)
    gs, gc = [], []
    for s0, c0 in zip(cells["start"][cells["leaf"]], cells["count"][cells["leaf"]]):
        for j in range(0, int(c0), 64):
            gs.append(s0 + j)
            gc.append(min(64, int(c0) - j))
    L = max(np.ptp(ps.x), np.ptp(ps.y), np.ptp(ps.z))
    ref = np.empty((n, 3))
    ref[o] = np.stack(orc.tree_gravity(ps.x[o], ps.y[o], ps.z[o], ps.m[o], t, L, 0.8, 1.0, 0.01, np.array(gs),
                                       np.array(gc))[:3], axis=1)
    d = np.linalg.norm(g - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert np.quantile(d, 0.99) <= 1e-9 and d.max() <= 1e-2, (np.quantile(d, 0.99), d.max())


def test_moments_of_a_large_ensemble(orc):
    """The same with 400 sets, whose first three levels are refined whatever they hold: lists (boxes and largest h of
    the nodes) of some sets exact, their gravity near the direct sum."""
    from gpu_helpers import gpu_gravity, gpu_neighbors
    sets, per = 400, 701
    n = sets * per
    ps = uniform_random(n, seed=105, h=(0.02, 0.1))
    ps.seg_offsets = np.arange(sets + 1, dtype=np.int64) * per
    ctx = make_ctx(n, sets, theta=0.6, G=1.0, soft_eps=0.05, nbr_capacity=512)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, n)
    got = np.stack(gpu_gravity(ctx, n))
    for i in range(0, n, 57 * per):
        x, y, z, m, h = (getattr(ps, f)[i:i + per] for f in ("x", "y", "z", "m", "h"))
        csr = orc.neighbors(x, y, z, h)
        assert np.array_equal(np.diff(off[i:i + per + 1]), np.diff(csr[0]))
        assert np.array_equal(idx[off[i]:off[i + per]] - i, csr[1])
        ref = np.stack(orc.gravity_direct(x, y, z, m, 1.0, 0.05)[:3])
        d = np.sqrt(((got[:3, i:i + per] - ref) ** 2).sum(0)) / np.sqrt((ref ** 2).sum(0))
        assert np.sqrt((d ** 2).mean()) <= 1e-2


# ---------------------------------------------------------------------------- CSR rows of short lists
@pytest.mark.parametrize("group", [8, 16, 64])
@pytest.mark.parametrize("n,mean", [(2001, 6), (2001, 10), (40_001, 3), (70_001, 6), (70_001, 30)])
def test_csr_of_short_lists(orc, n, mean, group):
    """Groups whose longest list has up to 8, up to 16 and more entries, by workgroups of four wavefronts and of one;
    a few groups of one set are long."""
    from gpu_helpers import gpu_neighbors
    h0 = (mean / (n * 32.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
    ps = uniform_random(n, seed=106, h=(0.7 * h0, 1.3 * h0))
    ps.x[:300], ps.y[:300], ps.z[:300] = (0.5 + 0.3 * h0 * np.random.default_rng(107).uniform(-1, 1, (3, 300)))
    ctx = make_ctx(n, group_size=group, nbr_capacity=1024)
    gpu_keys_order(ctx, parts(ps))
    off, idx = gpu_neighbors(ctx, n)
    ref = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    assert np.array_equal(off, ref[0]) and np.array_equal(idx, ref[1])


# ---------------------------------------------------------------------------- pair sums over long lists
@pytest.mark.parametrize("cap", [192, 193])
@pytest.mark.parametrize("n", [4097, 16384, 16385])
def test_pair_sums_by_list_capacity(orc, n, cap):
    """Groups of 8 take workgroups of 128 or 256 threads by the number of groups and the lists' capacity: FP64
    density and forces at both sides of each limit, 1e-12 of the sum of the terms' magnitudes."""
    from gpu_helpers import gpu_forces
    h0 = (40.0 / (n * 32.0 / 3.0 * np.pi)) ** (1.0 / 3.0)
    ps = uniform_random(n, seed=108, h=(0.5 * h0, 1.2 * h0))
    ctx = make_ctx(n, group_size=8, nbr_capacity=cap)
    gpu_keys_order(ctx, parts(ps))
    rho, P, c, hn = gpu_density(ctx, n)
    csr = orc.neighbors(ps.x, ps.y, ps.z, ps.h)
    for a, b in zip((rho, P, c, hn), orc.density(ps.fields(), csr)):
        assert np.max(np.abs(a - b) / np.abs(b)) <= 1e-12
    ax, ay, az, du = gpu_forces(ctx, n)
    r_ax, r_ay, r_az, r_du, Sa, Su = orc.forces(ps.fields(), rho, P, c, csr)
    assert np.all(np.sqrt((ax - r_ax) ** 2 + (ay - r_ay) ** 2 + (az - r_az) ** 2) <= 1e-12 * Sa)
    assert np.all(np.abs(du - r_du) <= 1e-12 * Su)


# ---------------------------------------------------------------------------- quadrupole walk, every form
@pytest.mark.parametrize("group", [8, 16, 32, 64])
def test_gravity_forms_against_the_walk(orc, group):
    """5,000 particles by one wavefront a group (8), two (16) and four (32, 64; FP32C two): FP64 against the oracle's
    walk over the same groups, 99% to 1e-9 (the rest where a borderline opening decision flips), and FP32C
    against FP64, whose decisions it shares, within FP32 rounding."""
    from gpu_helpers import gpu_gravity
    from workloads import polytrope_n1
    ps = polytrope_n1(5000, seed=109)
    ps.m = np.random.default_rng(110).uniform(0.5, 1.5, ps.n) / ps.n
    res = []
    for prec in (0, 1):
        ctx = make_ctx(ps.n, theta=0.5, G=1.0, soft_eps=0.01, precision=prec, leaf_size=16, group_size=group)
        k, o = gpu_keys_order(ctx, parts(ps))
        res.append(np.stack(gpu_gravity(ctx, ps.n), axis=1))
        ctx.close()
    cells = orc.octree(k[o], 4 * group)
    gs, gc = [], []
    for s0, c0 in zip(cells["start"][cells["leaf"]], cells["count"][cells["leaf"]]):
        for j in range(0, int(c0), group):
            gs.append(s0 + j)
            gc.append(min(group, int(c0) - j))
    L = max(np.ptp(ps.x), np.ptp(ps.y), np.ptp(ps.z))
    ref = np.empty((ps.n, 4))
    ref[o] = np.stack(orc.tree_gravity(ps.x[o], ps.y[o], ps.z[o], ps.m[o], orc.octree(k[o], 16), L, 0.5, 1.0, 0.01,
                                       np.array(gs), np.array(gc)), axis=1)
    gm = np.linalg.norm(ref[:, :3], axis=1)
    d, dp = np.linalg.norm(res[0][:, :3] - ref[:, :3], axis=1) / gm, np.abs(res[0][:, 3] / ref[:, 3] - 1.0)
    assert np.quantile(d, 0.99) <= 1e-9 and d.max() <= 1e-3 and np.quantile(dp, 0.99) <= 1e-9
    d, dp = np.linalg.norm(res[1][:, :3] - res[0][:, :3], axis=1) / gm, np.abs(res[1][:, 3] / res[0][:, 3] - 1.0)
    assert np.median(d) <= 2e-7 and d.max() <= 1e-5
    assert np.median(dp) <= 1e-7 and dp.max() <= 1e-6


# ---------------------------------------------------------------------------- sorts, every pass
def _points(n, copies):
    """Random points, each `copies` times, at random places of the input: ties across tiles and runs."""
    ps = uniform_random(n, seed=111 + n % 97, h=1e-4)
    k = np.random.default_rng(n).permutation(n) // copies
    for f in ("x", "y", "z", "vx", "vy", "vz"):
        setattr(ps, f, np.ascontiguousarray(getattr(ps, f)[k]))
    return ps


@pytest.mark.parametrize("n", [40_961, 524_289, 1_600_003, 2_200_003])
def test_step_sort_ties_in_every_pass(orc, n):
    """Tiles of 1,024 keys and passes of 8 and 8 ways; of 4,096 and 4, 4, 4, 4; and 4, 4, 4, 4, 2; and ten
    of 2: the step's sort, from the previous key order, with equal keys (16 particles a point) in the order of the IDs."""
    import torch
    import paper_2007_03097_amd as sph
    from gpu_helpers import to_np
    ps = _points(n, 16)
    ctx = make_ctx(n, nbr_capacity=64)
    pa = parts(ps, with_accel=True)
    keys = torch.zeros(n, dtype=torch.int64, device="cuda")
    order = torch.zeros(n, dtype=torch.int64, device="cuda")
    for flags in (sph.SPH_STEP_PRIMED, sph.SPH_STEP_RESUME):
        sph.sph_step(ctx.h, pa, 0.3, 1, flags)   # far enough to mix the order
        sph.sph_key_order(ctx.h, keys, order)
        k = to_np(keys).view(np.uint64)
        assert np.array_equal(k, orc.keys(*(to_np(pa[f]) for f in ("x", "y", "z"))))
        assert np.array_equal(to_np(order), orc.order(k))
        assert np.unique(k).size < n
    ctx.close()


@pytest.mark.parametrize("copies", [1, 16])
@pytest.mark.parametrize("n", [1_600_003, 2_200_003])
def test_caller_sort_of_large_sets(orc, n, copies):
    """Two-way passes over runs of like length, keys in any order, equal keys by index."""
    ps = _points(n, copies)
    ctx = make_ctx(n, nbr_capacity=16)
    k, o = gpu_keys_order(ctx, parts(ps))
    assert np.array_equal(k, orc.keys(ps.x, ps.y, ps.z)) and np.array_equal(o, orc.order(k))
    ctx.close()
