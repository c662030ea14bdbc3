"""GPU tests of single kernels at the sizes where they can go wrong, against the oracle."""
import numpy as np
import pytest

from workloads import uniform_random

from gpu_helpers import gpu_keys_order, make_ctx, parts, to_np

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
