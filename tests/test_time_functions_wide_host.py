"""Host emulation of the time functions' series (td4_device.hpp) where the
resolution is wide: the rule that admits an event to the series, read from the
source (r = max(|x|, |y|) G (|t| + s3), s3 the fit's constant), has to keep out
the events whose terms' rounding errors it would add up.  The terms' recurrence
multiplies by v = G u, u = G s^2 - t, which for a resolution of w lifetimes
exceeds what the terms themselves grow by w^2; the series' error stays a few
units as long as |v| max(|x|, |y|) is bounded by r."""
import math
import os
import re

import numpy as np
import pytest

from tests.test_time_functions_host import MAX, TEN, h_exact, series

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_1710_08826_amd", "csrc", "td4_device.hpp")
S3 = re.search(r"k\.s3 = (.*);", open(SRC).read()).group(1)


def s3(G, s):
    return eval(S3, {"G": G, "s": s, "fmax": max, "s2": s * s})


@pytest.mark.parametrize("w", [0.1, 1.0, 3.0, 5.0, 10.0, 20.0, 30.0, 100.0])
def test_series_of_admitted_events(w):
    rng = np.random.default_rng(5)
    G = 1.0 / 0.41
    s = w / G
    seen = 0
    for n_max, line in ((10, TEN), (20, MAX)):
        for f in (0.999, 0.7, 0.3):
            d = line * f / (3.0 * w)  # the size at which times about zero reach f of the line with s3 = 3 s
            tmax = line / (d * G) - s3(G, s)
            if tmax <= 0:
                continue
            t = np.concatenate([rng.uniform(-tmax, tmax, 1000), [0.0, tmax, -tmax]])
            t = t[(np.abs(t) < 8 * s) & (t < 25.0 / G)]
            seen += t.size
            for x, y in ((d, -0.6 * d), (0.3 * d, d)):
                h0, Hc, Hs, hr, hi = series(G, s, x, y, t, n_max)
                hp, hm = (h_exact(complex(G * (1 - q), 0.0), t, s).real for q in (y, -y))
                hc = h_exact(complex(G, -G * x), t, s)
                for v, e in ((Hc, 0.5 * (hp + hm)), (Hs, 0.5 * (hp - hm)), (hr, hc.real), (hi, hc.imag)):
                    # as in the emulation over ordinary resolutions
                    assert np.max(np.abs(v - e) / h0) < 2e-14
    assert seen > 0 or w > 3.0


def test_rule_bounds_the_recurrence():
    """r >= |v| max(|x|, |y|) for times at which the recurrence cancels (u > 0), and r is what it was for resolutions up to 3 tau."""
    rng = np.random.default_rng(6)
    for _ in range(2000):
        G, w = 10.0 ** rng.uniform(-2, 2), 10.0 ** rng.uniform(-3, 2.5)
        s = w / G
        t = rng.uniform(-9, 9) * s
        u = G * s * s - t
        if u > 0.0:
            assert abs(t) + s3(G, s) >= u * (1 - 1e-15)
        if w <= 3.0:
            assert math.isclose(s3(G, s), 3.0 * s, rel_tol=1e-15)
