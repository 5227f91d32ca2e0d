"""Density of a three-body model to the last bits: far from a resonance of no
width |A|^2 is 1/(m0^2 - s)^2, so the density times that denominator is one
number for all events, up to the roundings of the amplitude (one resonance: the
mass difference, the denominator, its reciprocal, the amplitude's two products
and two squares, the quotient by the normalization: 14 units of 2^-53 at most,
either way between two events; four equal ones: three more sums in the square)."""
import numpy as np
import pytest

import synth
from oracle import dalitz3 as OD
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

M0, W0 = 0.892, 1e-7


@pytest.mark.parametrize("free", [False, True])
@pytest.mark.parametrize("copies,units", [(1, 14), (4, 20)])
def test_reciprocals(copies, units, free):
    from paper_1710_08826_amd import Model
    say("density rounding", copies, free)
    d = OD.config1_desc(grid=(64, 64), free_lineshapes=free, resonances=(("12", 0, M0, W0, (1.0, 0.0)),) * copies)
    th = np.tile([1.0, 0.0], copies)
    if free:
        th = np.concatenate([th, np.tile([M0, W0], copies)])
    ev = synth.dalitz_events(20000, seed=91)
    s = ev[0].astype(np.longdouble)
    a = np.longdouble(M0 * M0) - s
    keep = np.abs(a) > 0.02  # the width's part of the denominator, (m0 w0 / a)^2 < 3e-11, has its own error of 1e-14
    m1, m2 = (float(v) for v in d["m"][:2])
    q = lambda x: np.sqrt((x - (m1 + m2) ** 2) * (x - (m1 - m2) ** 2)) / (2.0 * np.sqrt(x))
    b = W0 * M0 * M0 / q(M0 * M0) * q(ev[0]) / np.sqrt(ev[0])
    p = Model(d).eval(th, to_dev(ev)).cpu().numpy().astype(np.longdouble)
    r = (p * (a * a + b.astype(np.longdouble) ** 2))[keep]
    assert keep.sum() > 15000
    spread = float(r.max() / r.min() - 1)
    assert spread <= 2 * units * 2.0 ** -53, spread / 2.0 ** -53
