"""Time-dependent three-body models whose resonances share lineshapes in every
way the pass distinguishes: twins in the two charged pairs in either order,
repeated ones within a pair, the same numbers with another spin (not shared),
one without a twin, and the charge-symmetric pair; against the oracle.  Also
azimuths far outside their domain in the four-body model (the sine's and
cosine's reduction and their library fallback)."""
import numpy as np
import pytest

import synth
from oracle import td4 as OT, tddp3 as T
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

TABLES = {
    "twins, later pair first": (("13", 1, 0.7753, 0.1491, (0.6, 0.1)), ("12", 1, 0.7753, 0.1491, (1.0, 0.0)),
                                ("13", 1, 0.7753, 0.1491, (0.2, -0.1)), ("23", 0, 0.99, 0.07, (0.1, 0.05))),
    "another spin, no twin": (("12", 1, 1.465, 0.4, (1.0, 0.0)), ("13", 0, 1.465, 0.4, (0.3, 0.2)),
                              ("12", 2, 1.3, 0.11, (0.2, 0.1)), ("13", 2, 1.3, 0.12, (0.2, -0.1))),
    "symmetric pair only": (("23", 1, 0.7753, 0.1491, (1.0, 0.0)), ("23", 1, 0.7753, 0.1491, (0.4, 0.3)),
                            ("23", 2, 1.2755, 0.1867, (0.2, -0.1)), ("23", 0, 0.5, 0.4, (0.2, 0.1))),
    "one": (("13", 0, 0.99, 0.07, (1.0, 0.0)),),
}


@pytest.mark.parametrize("name", sorted(TABLES))
def test_shared_lineshapes(name):
    from paper_1710_08826_amd import Model
    say("tddp3 shared lineshapes:", name)
    res = TABLES[name]
    d = T.pipipi0_desc(grid=(64, 64), resonances=res)
    m = Model(d)
    ev = synth.tddp3_events(1500, seed=49)
    th = T.truth_theta(resonances=res, x=0.02, y=0.03)
    k = 2 * len(res)
    th[k:2 * k] = th[k:2 * k] * 0.9 + 0.05
    v, g = m.nll(th, to_dev(ev), grad=True)
    vo, go = T.nll_grad(th, ev, d)
    assert rel_close(v, vo, 1e-12), (v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, r


@pytest.mark.parametrize("turns", [1, 10_000, 30_000])
def test_azimuth_outside_its_domain(turns):
    from paper_1710_08826_amd import Model
    say("td4 azimuth", turns)
    d = synth.td4_desc()
    mc = synth.td4_phase_space(2000, seed=41)
    m = Model(d)
    m.set_norm_sample(to_dev(mc))
    ev = synth.td4_events(600, seed=50)
    ev[4, ::5] += 2.0 * np.pi * turns
    ev[4, 1::7] -= 2.0 * np.pi * turns
    th = synth.td4_truth()
    v, g = m.nll(th, to_dev(ev), grad=True)
    vo, go = OT.nll_grad(th, ev, mc, d)
    assert rel_close(v, vo, 1e-12), (v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, r
