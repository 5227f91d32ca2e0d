"""The density of an event does not depend on the other events of the call: the
same bits alone, in a full sample and in any order, where the events take
different forms of the time functions (r = max(|x|, |y|) G (|t| + 3 s) on both
sides of 1/8 and of 5/4) and of the azimuth's sine and cosine."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("xy", [(0.004, 0.006), (0.05, -0.04), (-0.2, 0.1), (0.8, 0.3)])
def test_td4(xy):
    from paper_1710_08826_amd import Model
    say("density of events alone", xy)
    d, th = synth.td4_desc(), synth.td4_truth()
    th[-2:] = xy
    m = Model(d)
    m.set_norm_sample(to_dev(synth.td4_phase_space(2000, seed=62)))
    n = 520
    ev = synth.td4_events(n, seed=64)
    g, s = 1.0 / d["tau"], d["sigma_t"]
    ev[5] = np.random.default_rng(6).uniform(-4 * s, 14.0 / g, n)
    ev[4, 40] += 2.0e5 * np.pi
    evd = to_dev(ev)
    p = m.eval(th, evd)
    order = torch.from_numpy(np.random.default_rng(7).permutation(n)).cuda()
    assert torch.equal(m.eval(th, evd[:, order].contiguous()), p[order])
    for i in range(0, 130):
        assert torch.equal(m.eval(th, evd[:, i:i + 1]), p[i:i + 1]), i
