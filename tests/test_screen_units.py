"""The list kernel's screen in units of the group's reach, emulated on the CPU as in test_matrix_screen: with lengths
times k, the power of two near 1 / (2 R + hg), it decides the same pairs whatever unit the input is in, and
in the input's own unit it would decide none of them outside the FP32 range."""
import numpy as np
import pytest

from test_matrix_screen import _screen


def _unit(reach):
    return 2.0 ** (-np.floor(np.log2(reach)))


@pytest.mark.parametrize("unit", [2.0 ** -300, 2.0 ** -60, 2.0 ** 75, 2.0 ** 300])
def test_same_pairs_decided_in_any_unit(unit):
    rng = np.random.default_rng(19)
    s, n = 1.0 / 56, 50_000
    lo = np.array([0.2, 0.05, 0.05])
    hi = lo + 4 * s
    ta = rng.uniform(lo, hi, size=(n, 3))
    sb = ta + rng.uniform(-3 * s, 3 * s, size=(n, 3))
    ha, hb = rng.uniform(0.6 * s, 1.2 * s, n), rng.uniform(0.6 * s, 1.2 * s, n)
    hg, hm = 1.2 * s, 1.2 * s
    ref = None
    for u in (1.0, unit):
        o = 0.5 * (lo + hi) * u
        k = _unit(2 * np.sqrt(((hi * u - o) ** 2).sum()) + hg * u)
        with np.errstate(over="ignore", invalid="ignore", under="ignore"):
            D, M, und = _screen(ta * (u * k), sb * (u * k), ha * (u * k), hb * (u * k), lo * (u * k), hi * (u * k), hg * u * k,
                                hm * u * k, "")
            assert np.isfinite(M) and und.mean() < 1e-3
            if ref is None:
                ref = D
            assert np.array_equal(ref, D)
            if u != 1.0:    # the input's own unit: the margin swallows everything, or there is none
                _, M1, und1 = _screen(ta * u, sb * u, ha * u, hb * u, lo * u, hi * u, hg * u, hm * u, "")
                assert not M1 < 2.0 ** 100 or und1.all() or M1 > (hg * u) ** 2
