"""Density per event at the edges of a workgroup: one event, one less and one
more than a workgroup, several; from a view of a larger sample (leading
dimension above the size), against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import common
from oracle import dalitz3 as OD
from oracle import td4 as OT
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

SIZES = [1, 255, 256, 257, 1500]


@pytest.mark.parametrize("free", [False, True])
def test_dalitz(free):
    from paper_1710_08826_amd import Model
    d = OD.config1_desc(grid=(64, 64), free_lineshapes=free)
    th = OD.truth_theta(d)
    m, om = Model(d), OD.Dalitz(d)
    ev = synth.dalitz_events(max(SIZES) + 9, seed=61)
    with torch.no_grad():
        ref = om.density_unnorm(common.as_t(th), common.as_t(ev[0]), common.as_t(ev[1])).numpy()
    ref = ref / OD.norm_value(om, th, om.grid_cells())
    evd = to_dev(ev)
    for n in SIZES:
        say("density dalitz", free, n)
        p = m.eval(th, evd[:, :n]).cpu().numpy()
        # relative to each density, which interference can leave far below its terms
        assert p.shape == (n,) and np.allclose(p, ref[:n], rtol=1e-11, atol=1e-13 * ref.max())


def test_td4():
    from paper_1710_08826_amd import Model
    d, th = synth.td4_desc(), synth.td4_truth()
    mc = synth.td4_phase_space(2000, seed=62)
    m, om = Model(d), OT.TD4(d)
    m.set_norm_sample(to_dev(mc))
    ev = synth.td4_events(max(SIZES) + 9, seed=63)
    with torch.no_grad():
        ref = om.rate(torch.tensor(th), torch.tensor(ev)).numpy()
        I = common.fsum(om.integrated_rate(torch.tensor(th), torch.tensor(mc))) / mc.shape[1]
    ref = ref / I
    evd = to_dev(ev)
    for n in SIZES:
        say("density td4", n)
        p = m.eval(th, evd[:, :n]).cpu().numpy()
        # the time functions carry 1e-13 of their largest value (t far before zero: absolute)
        assert p.shape == (n,) and np.allclose(p, ref[:n], rtol=1e-11, atol=1e-13 * ref.max())
