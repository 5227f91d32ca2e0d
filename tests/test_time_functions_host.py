"""Host emulation of the device's time functions (td4_device.hpp): the
polynomial of exp(y^2) erfc(y) with the coefficients of td4_types.hpp, and the
Taylor series of h(a; t) about a = G with ten and with twenty terms, against
SciPy's Faddeeva function over the resolutions, times and mixing parameters
each form is taken for."""
import math
import os
import re

import numpy as np
from scipy.special import erfcx, wofz

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_1710_08826_amd", "csrc", "td4_types.hpp")
TEXT = open(SRC).read()
WE = [float.fromhex(v) for v in re.findall(r"-?0x1\.[0-9a-f]+p[-+]\d+", TEXT[TEXT.index("#define FN_ERFC_COEFFS"):])]
K = float(re.search(r"kErfcK = ([\d.]+);", TEXT).group(1))
TEN = float(re.search(r"kTimeSeriesTen = ([\d.]+);", TEXT).group(1))
MAX = float(re.search(r"kTimeSeriesMax = ([\d.]+);", TEXT).group(1))


def erfcx_pos(y):
    i = 1.0 / (K + y)
    z = (K - y) * i
    p = np.full_like(z, WE[-1])
    for a in reversed(WE[:-1]):
        p = p * z + a
    return p * i


def test_erfcx_polynomial():
    assert len(WE) == 24
    rng = np.random.default_rng(3)
    y = np.concatenate([[0.0], 10.0 ** rng.uniform(-8, 4, 20000), rng.uniform(0, 10, 20000)])
    # SciPy's own error (below 1e-15) and the polynomial's rounding (24 steps whose partial sums stay within
    # twice the result: a few units)
    assert np.max(np.abs(erfcx_pos(y) / erfcx(y) - 1.0)) < 2e-15


def h_exact(a, t, s):
    """1/2 exp(a^2 s^2/2 - a t) erfc((a s^2 - t)/(s sqrt 2)), complex a, through w(z)."""
    z = (a * s * s - t) / (s * math.sqrt(2.0))
    g = np.exp(-t * t / (2 * s * s))
    up = 0.5 * g * wofz(1j * np.where(z.real >= 0, z, -z))
    return np.where(z.real >= 0, up, np.exp(0.5 * a * a * s * s - a * t) - up)


def series(G, s, x, y, t, n_max):
    g, u = np.exp(-t * t / (2 * s * s)), G * s * s - t
    z = u / (s * math.sqrt(2.0))
    e = 0.5 * g * erfcx_pos(np.abs(z))
    c = [np.where(z >= 0, e, np.exp(0.5 * G * G * s * s - G * t) - e)]
    v, w = G * u, (G * s) ** 2
    c.append(v * c[0] - G * s / math.sqrt(2 * math.pi) * g)
    for n in range(2, n_max + 1):
        c.append((v * c[n - 1] + w * c[n - 2]) / n)
    Hc = sum(c[n] * y ** n for n in range(0, n_max + 1, 2))
    Hs = -sum(c[n] * y ** n for n in range(1, n_max + 1, 2))
    hr = sum((-1) ** (n // 2) * c[n] * x ** n for n in range(0, n_max + 1, 2))
    hi = -sum((-1) ** (n // 2) * c[n] * x ** n for n in range(1, n_max + 1, 2))
    return c[0], Hc, Hs, hr, hi


def test_series_against_the_functions_themselves():
    rng = np.random.default_rng(4)
    for n_max, line in ((10, TEN), (20, MAX)):
        for _ in range(40):
            G, s = 10.0 ** rng.uniform(-1, 1), 10.0 ** rng.uniform(-3, -0.5)
            d = 10.0 ** rng.uniform(-3, -0.6)
            x, y = d * rng.choice([1.0, 0.3, 0.0]), -d * rng.choice([1.0, 0.6])
            tmax = min(line / (max(abs(x), abs(y)) * G) - 3 * s, 25.0 / G)
            if tmax <= 0:
                continue
            t = np.concatenate([rng.uniform(-5 * s, tmax, 500), [tmax, 0.0]])
            t = t[np.abs(t) <= tmax]
            h0, Hc, Hs, hr, hi = series(G, s, x, y, t, n_max)
            hp, hm = (h_exact(complex(G * (1 - q), 0.0), t, s).real for q in (y, -y))
            hc = h_exact(complex(G, -G * x), t, s)
            # both sides' roundings: the exponent G t (up to 25) rounds to a few 1e-15 in each of them
            for v, e in ((Hc, 0.5 * (hp + hm)), (Hs, 0.5 * (hp - hm)), (hr, hc.real), (hi, hc.imag)):
                assert np.max(np.abs(v - e) / h0) < 2e-14
