"""The neighbour kernel's matrix-core screen, emulated on the CPU: whenever it decides a pair (D' < 0 or
D' > 2M), the decision is that of the FP64 predicate fl(fl(fl(dx dx) + fl(dy dy)) + fl(dz dz)) < fl(t t).

D' = a . 2b + h_a 2h_b + c_b + (c_a + M) in FP32, offsets a, b from the centre of the group's box and
h formed in FP64 and rounded once, c = h^2 - |x|^2 in FP64 rounded once; M = 2^-19 (R^2 + t^2) + 2^-100
with R = 2 (half diagonal) + hg + hm, t = hg + hm.  The order and rounding of the six accumulations are the
hardware's, so several are tried: fused in either order, products rounded first, pairs first, and every
operation truncated toward zero instead of rounded."""
import numpy as np
import pytest

f32, f64 = np.float32, np.float64


def _rne(x):
    return x.astype(f32)


def _trunc(x):
    y = x.astype(f32)
    over = np.abs(y.astype(f64)) > np.abs(x)
    return np.where(over, np.nextafter(y, f32(0)), y).astype(f32)


def _accumulate(terms, how):
    """terms: list of (p, q) FP32 pairs, accumulated by the given scheme."""
    rnd = _trunc if "trunc" in how else _rne
    prod = [p.astype(f64) * q.astype(f64) for p, q in terms]   # exact in FP64
    if "reverse" in how:
        prod = prod[::-1]
    if "round" in how:
        prod = [rnd(x).astype(f64) for x in prod]
    if "pairs" in how:
        prod = [rnd(prod[i] + prod[i + 1]).astype(f64) for i in range(0, 6, 2)]
    acc = np.zeros_like(prod[0])
    for x in prod:
        acc = rnd(acc + x).astype(f64)
    return acc.astype(f32)


def _screen(ta, sb, ha, hb, lo, hi, hg, hm, how):
    o = 0.5 * (lo + hi)
    half = np.sqrt((np.maximum(hi - o, o - lo) ** 2).sum())
    up = 1 + 2.0 ** -20
    reach, hgf, hmf = f32((2 * half + hg) * up), f32(hg * up), f32(hm)
    R, tt = f32(reach + hmf), f32(hgf + hmf)
    M = f32(f64(f32(f64(R) * R + f64(f32(tt * tt)))) * (2.0 ** -19 * (1 + 2.0 ** -18)) + 2.0 ** -100)
    a, b = ta - o, sb - o
    ca, cb = f32(ha * ha - (a * a).sum(1)), f32(hb * hb - (b * b).sum(1))
    a, b = a.astype(f32), (f32(2) * b.astype(f32)).astype(f32)
    one = np.ones(len(ha), f32)
    terms = [(a[:, 0], b[:, 0]), (a[:, 1], b[:, 1]), (a[:, 2], b[:, 2]),
             (ha.astype(f32), (f32(2) * hb.astype(f32)).astype(f32)), (one, cb), ((ca + M).astype(f32), one)]
    D = _accumulate(terms, how)
    lim = f32(f32(2) * M * f32(1 + 2.0 ** -18))
    return D, M, (D >= 0) & (D <= lim)


@pytest.mark.parametrize("how", ["", "reverse", "round", "round pairs", "trunc", "trunc reverse", "trunc round pairs"])
def test_decided_pairs_are_exact(how):
    rng = np.random.default_rng(17)
    seen_decided = seen_undecided = 0
    for scale, origin in ((1e-3, 0.3), (1.0, 10.0), (1e-6, 1.0), (1e5, -3e5), (3e-2, 0.0), (1e-13, 0.0), (1e12, 1e13)):
        n = 60_000
        lo = origin + rng.uniform(-1, 1, size=3) * scale
        hi = lo + scale * rng.uniform(0.1, 4.0, size=3)
        ta = rng.uniform(lo, hi, size=(n, 3))
        dirn = rng.normal(size=(n, 3))
        dirn /= np.linalg.norm(dirn, axis=1, keepdims=True)
        r = scale * 10.0 ** rng.uniform(-1, 0.5, size=n)
        sb = ta + dirn * r[:, None]
        dist = np.sqrt(((ta - sb) ** 2).sum(1))
        rel = np.where(rng.random(n) < 0.25, rng.integers(-8, 9, size=n) * 2.0 ** -52,
                       np.sign(rng.normal(size=n)) * 10.0 ** rng.uniform(-12, -1, size=n))
        ha = 0.5 * dist * (1 + rel) * rng.uniform(0.3, 1.0, size=n)
        hb = dist * (1 + rel) - ha
        hg, hm = ha.max(), hb.max()
        gap = np.maximum(0, np.maximum(sb - hi, lo - sb))
        near = (gap ** 2).sum(1) < (hg + hb) ** 2        # the group-box filter
        ta, sb, ha, hb = ta[near], sb[near], ha[near], hb[near]
        D, M, und = _screen(ta, sb, ha, hb, lo, hi, hg, hm, how)
        d = ta - sb
        exact = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2] < (ha + hb) * (ha + hb)
        assert np.array_equal((D >= 0)[~und], exact[~und])
        delta = (ha + hb) ** 2 - (d * d).sum(1)          # the margin is about twice the error
        assert np.abs(D.astype(f64) - f64(M) - delta).max() <= 0.55 * M
        seen_decided += int((~und).sum())
        seen_undecided += int(und.sum())
    assert seen_decided > 50_000 and seen_undecided > 50_000   # both paths exercised


def test_ordinary_pairs_are_decided():
    rng = np.random.default_rng(18)
    s, n = 1.0 / 56, 200_000
    lo = np.array([0.2, 0.05, 0.05])
    ta = rng.uniform(lo, lo + 4 * s, size=(n, 3))
    sb = ta + rng.uniform(-3 * s, 3 * s, size=(n, 3))
    h = np.full(n, 1.2 * s)
    D, M, und = _screen(ta, sb, h, h, lo, lo + 4 * s, 1.2 * s, 1.2 * s, "")
    assert und.mean() < 1e-3
