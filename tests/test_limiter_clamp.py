"""The FP64 monotonised-central limiter is a clamp of the quarter sum of the
two differences to the interval from 0 to the one of smaller magnitude; it is
the select form up to the sign of a zero (halving and doubling are exact), and
a NaN difference yields a finite value as the select form's 0 does."""
import numpy as np
import pytest


def clamp_form(dp, dm):
    lo, hi = np.fmin(np.fmax(dp, dm), 0.0), np.fmax(np.fmin(dp, dm), 0.0)
    return 2.0 * np.fmax(np.fmin(0.25 * (dp + dm), hi), lo)


def select_form(dp, dm):
    c = 0.5 * (dp + dm)
    m = np.fmin(np.fmin(np.abs(c), 2.0 * np.abs(dp)), 2.0 * np.abs(dm))
    return np.where(dp * dm > 0.0, np.copysign(m, c), 0.0)


@pytest.mark.parametrize("scale", [1e-140, 1e-9, 1.0, 1e9, 1e140])
def test_clamp_is_the_limiter(scale):
    rng = np.random.default_rng(11)
    dp, dm = scale * rng.standard_normal((2, 200000)) * 10.0 ** rng.uniform(-3, 3, (2, 200000))
    edge = np.array([0.0, -0.0, scale, -scale, 3.0 * scale, -3.0 * scale])
    dp, dm = np.concatenate([dp, np.repeat(edge, 6)]), np.concatenate([dm, np.tile(edge, 6)])
    assert np.array_equal(clamp_form(dp, dm), select_form(dp, dm))


def test_non_finite_differences():
    for a in (1.0, -1.0, 0.0):
        assert np.isfinite(clamp_form(np.nan, a)) and np.isfinite(clamp_form(a, np.nan))
    assert clamp_form(np.inf, 1.0) == select_form(np.inf, 1.0) == 2.0
    assert clamp_form(-np.inf, -1.0) == select_form(-np.inf, -1.0) == -2.0
    assert clamp_form(np.inf, -1.0) == select_form(np.inf, -1.0) == 0.0
