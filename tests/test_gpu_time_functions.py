"""The time functions' forms on the device -- ten series terms, twenty, and
the three functions one by one -- against the oracle: mixing parameters and
decay times on both sides of the lines between them (r = max(|x|, |y|) G
(|t| + 3 s) at 1/8 and 5/4), waves that hold events of one side only and of
both, times below zero.  Tolerances are those of the models' own parity tests
(NLL 1e-12, gradient 1e-10)."""
import numpy as np
import pytest

import synth
from oracle import td4 as OT, tddp3 as T
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

N = 700
MIXING = [(0.0, 0.0), (0.004, 0.006), (0.05, -0.04), (-0.2, 0.1)]


def times(g, s, xy, line):
    """Decay times around r = line (None: the whole range), and a few below zero."""
    d = max(abs(xy[0]), abs(xy[1]), 1e-3) * g
    rng = np.random.default_rng(5)
    if line is None:
        t = rng.uniform(-4 * s, 12.0 / g, N)
    else:
        t = np.clip((line / d - 3 * s) * rng.choice([0.999, 1.001, 1.0], N), 0.0, 14.0 / g)
    t[::97] = -rng.uniform(0, 4 * s, t[::97].size)
    return t


@pytest.mark.parametrize("line", [None, 0.125, 1.25])
@pytest.mark.parametrize("xy", MIXING)
def test_four_body(xy, line):
    from paper_1710_08826_amd import Model
    say("time functions td4", xy, line)
    d = synth.td4_desc()
    mc = synth.td4_phase_space(2000, seed=41)
    m = Model(d)
    m.set_norm_sample(to_dev(mc))
    ev = synth.td4_events(N, seed=47)
    ev[5] = times(1.0 / d["tau"], d["sigma_t"], xy, line)
    th = synth.td4_truth()
    th[-2:] = xy
    v, g = m.nll(th, to_dev(ev), grad=True)
    vo, go = OT.nll_grad(th, ev, mc, d)
    assert rel_close(v, vo, 1e-12), (v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, r
    assert rel_close(m.nll(th, to_dev(ev)), v, 1e-14)


@pytest.mark.parametrize("line", [None, 0.125, 1.25])
@pytest.mark.parametrize("xy", MIXING)
def test_three_body(xy, line):
    from paper_1710_08826_amd import Model
    say("time functions tddp3", xy, line)
    d = T.pipipi0_desc(grid=(64, 64))
    m = Model(d)
    ev = synth.tddp3_events(N, seed=48)
    ev[2] = times(1.0 / d["tau"], d["sigma_t"], xy, line)
    th = T.truth_theta(x=xy[0], y=xy[1])
    v, g = m.nll(th, to_dev(ev), grad=True)
    vo, go = T.nll_grad(th, ev, d)
    assert rel_close(v, vo, 1e-12), (v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, r
