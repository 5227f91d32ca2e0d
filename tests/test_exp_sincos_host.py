"""Host emulation of the passes' exponential, sine and cosine (fastmath.hpp):
the sequences with the coefficients of the source, every fused multiply-add
evaluated exactly and rounded once, against the C library (itself within one
unit) over the arguments the passes meet and the ends of their ranges."""
import math
import os
import random
import re
from fractions import Fraction

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_1710_08826_amd", "csrc", "fastmath.hpp")
TEXT = open(SRC).read()
HEX = r"(-?0x[0-9a-f.]+p[-+]\d+)"


def body(name):
    t = TEXT[TEXT.index(name):]
    return t[:t.index("\n}\n")]


def coefficients(name, var):
    b = body(name)
    return [float.fromhex(re.search(rf"double {var} = {HEX}", b).group(1))] + \
        [float.fromhex(v) for v in re.findall(rf"{var} = fma_sc\({var}, \w+, {HEX}\)", b)]


EXP, SIN, COS = coefficients("double exp_fast", "p"), coefficients("void sincos_fast", "s"), coefficients("void sincos_fast", "c")
LN2 = [float.fromhex(v) for v in re.findall(rf"kLn2\w+ = {HEX}", body("double exp_fast"))]
PIO2_LO, PIO2_HI = [float.fromhex(v) for v in re.findall(rf"fma\(-k, {HEX}", body("void sincos_fast"))]


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def horner(c, x):
    p = c[0]
    for a in c[1:]:
        p = fma(p, x, a)
    return p


def exp_fast(x):
    n = float(round(x * 1.44269504088896340736))
    r = fma(-n, LN2[1], fma(-n, LN2[0], x))
    p = horner(EXP, r)
    return math.ldexp(fma(fma(p, r, 1.0), r, 1.0), int(n))


def sincos_fast(x):
    k = float(round(x * 0.63661977236758134308))
    r = fma(-k, PIO2_LO, fma(-k, PIO2_HI, x))
    z = r * r
    s, c = fma(r * z, horner(SIN, z), r), fma(z * z, horner(COS, z), fma(z, -0.5, 1.0))
    q = int(k)
    a, b = (c, s) if q & 1 else (s, c)
    return (-a if q & 2 else a), (-b if (q + 1) & 2 else b)


def test_coefficients_read():
    assert (len(EXP), len(SIN), len(COS), len(LN2)) == (10, 6, 6, 2)


def test_exp():
    rng = random.Random(1)
    args = [rng.uniform(-40, 5) for _ in range(2000)] + [rng.uniform(-700, 700) for _ in range(1000)] + [0.0, 709.0, -708.0]
    args += [(k + 0.5) * math.log(2) * (1 + d) for k in (-3, -1, 0, 1, 7) for d in (-1e-15, 0.0, 1e-15)]
    for x in args:
        e = math.exp(x)
        # truncation 1.6e-17, two roundings of the last steps (1.5 units of 2^-53) and the C library's own unit
        assert abs(exp_fast(x) - e) <= 4e-16 * e, x


def test_sincos():
    rng = random.Random(2)
    args = [rng.uniform(-4, 4) for _ in range(2000)] + [rng.uniform(-1e5, 1e5) for _ in range(500)] + [0.0, 1e-300]
    args += [k * math.pi / 4 * (1 + d) for k in range(-9, 10) for d in (-1e-12, 0.0, 1e-12)]
    for x in args:
        s, c = sincos_fast(x)
        # below 2e-16 stated, the C library's half unit besides
        assert abs(s - math.sin(x)) <= 3.2e-16 and abs(c - math.cos(x)) <= 3.2e-16, x
