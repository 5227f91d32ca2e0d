"""Host emulation of the region predicate of the three-body event generators:
wherever the boundary polynomial decides (outside its band about the boundary),
it decides as the predicate through the bounds lo <= s23 <= hi does, for points
of the box, on the boundary and 1e-16 to 1e-3 away from it, for heavy, light,
massless and threshold-like daughters."""
import numpy as np
import pytest

MASSES = [(1.865, 0.494, 0.140, 0.135), (1.865, 0.140, 0.140, 0.135), (5.279, 0.494, 3.097, 0.140),
          (1.0, 0.0, 0.0, 0.0), (2.0, 0.0, 0.9, 0.3), (1.0, 0.33, 0.33, 0.33), (3.0, 1e-4, 1.0, 1.0)]


def exact(m, s12, s13):
    M2, m1, m2, m3 = (v * v for v in m)
    rs = np.sqrt(s12)
    e2 = (s12 - m1 + m2) / (2.0 * rs)
    e3 = (M2 - s12 - m3) / (2.0 * rs)
    p2 = np.sqrt(np.maximum(e2 * e2 - m2, 0.0))
    p3 = np.sqrt(np.maximum(e3 * e3 - m3, 0.0))
    es = e2 + e3
    s23 = (M2 + m1 + m2 + m3) - s12 - s13
    lo, hi = es * es - (p2 + p3) * (p2 + p3), es * es - (p2 - p3) * (p2 - p3)
    return (s23 >= lo) & (s23 <= hi), lo, hi


def quick(m, s12, s13):
    """(decided, inside); the products rounded where the device fuses them."""
    M2, m1, m2, m3 = (v * v for v in m)
    s23 = (M2 + m1 + m2 + m3) - s12 - s13
    A, B, f = s12 - m1 + m2, M2 - s12 - m3, 4.0 * s12
    a, b = A * A - f * m2, B * B - f * m3
    D = f * (s23 - m2 - m3) - 2.0 * A * B
    F = D * D - 4.0 * a * b
    ab = np.abs(A) + np.abs(B)
    T = f * (np.abs(s23) + m2 + m3) + ab * ab
    return (a > 0.0) & (b > 0.0) & (np.abs(F) > 1e-12 * T * T), F < 0.0


@pytest.mark.parametrize("m", MASSES)
def test_polynomial_decides_as_the_bounds(m):
    rng = np.random.default_rng(5)
    n = 200_000
    lo12, hi12 = (m[1] + m[2]) ** 2, (m[0] - m[3]) ** 2
    lo13, hi13 = (m[1] + m[3]) ** 2, (m[0] - m[2]) ** 2
    u = rng.random(n)
    edge = 10.0 ** rng.uniform(-16, 0, n)  # s12 near either end
    s12 = lo12 + (hi12 - lo12) * np.where(u < 0.6, rng.random(n), np.where(u < 0.8, edge, 1.0 - edge))
    s12 = np.maximum(s12, 1e-300)
    _, lo, hi = exact(m, s12, 0.0)
    total = sum(v * v for v in m)
    with np.errstate(all="ignore"):
        near = total - s12 - np.where(rng.random(n) < 0.5, lo, hi)  # s13 on the boundary
        away = near + np.where(rng.random(n) < 0.5, 1, -1) * 10.0 ** rng.uniform(-16, -3, n) * (hi13 - lo13)
        box = lo13 + (hi13 - lo13) * rng.random(n)
        share = 0.0
        for s13 in (box, near, away):
            want, _, _ = exact(m, s12, s13)
            decided, inside = quick(m, s12, s13)
            assert np.array_equal(inside[decided], want[decided])
            if s13 is box:
                share = np.mean(~decided[u < 0.6])
    assert share < 1e-4
