"""Time resolutions of several lifetimes up to thirty, where h(a; t) at a = G and
its derivatives differ by orders of magnitude: value and gradient of the mixing
models and the four-body density against the oracle, for mixing parameters whose
events take the series' ten terms, its twenty and the functions one by one.
Tolerances are those of the models' own parity tests (NLL 1e-12, gradient 1e-10);
the density's is the sum of the oracle's and the device's own roundings of the
three functions (each a few 1e-15 of the largest, ten of them in the rate)."""
import numpy as np
import pytest
import torch

import synth
from oracle import common
from oracle import td4 as OT, tddp3 as T
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

N = 700
WIDTHS = [3.0, 6.0, 12.0, 30.0]
# max(|x|, |y|) (|t| + 3 s) / tau for t near zero: the series' ten terms end at 1/8, its twenty at 5/4
REACH = [0.12, 0.6, 1.2, 8.0]


def mixing(w, reach):
    return reach / (3.0 * w + 2.0)


def times(tau, s, near):
    rng = np.random.default_rng(8)
    return rng.uniform(-2.0, 2.0, N) * tau if near else rng.normal(0.0, 1.0, N) * s


@pytest.mark.parametrize("near", [True, False])
@pytest.mark.parametrize("reach", REACH)
@pytest.mark.parametrize("w", WIDTHS)
def test_four_body(w, reach, near):
    from paper_1710_08826_amd import Model
    say("wide resolution td4", w, reach, near)
    d = mixing(w, reach)
    tau = synth.td4_desc()["tau"]
    desc = synth.td4_desc(sigma_t=w * tau)
    mc = synth.td4_phase_space(2000, seed=41)
    m, om = Model(desc), OT.TD4(desc)
    m.set_norm_sample(to_dev(mc))
    ev = synth.td4_events(N, seed=47)
    ev[5] = times(tau, w * tau, near)
    th = synth.td4_truth()
    th[-2:] = (d, -0.6 * d)
    v, g = m.nll(th, to_dev(ev), grad=True)
    vo, go = OT.nll_grad(th, ev, mc, desc)
    assert rel_close(v, vo, 1e-12), (v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, r
    with torch.no_grad():
        ref = om.rate(torch.tensor(th), torch.tensor(ev)).numpy()
        I = common.fsum(om.integrated_rate(torch.tensor(th), torch.tensor(mc))) / mc.shape[1]
    ref = ref / I
    p = m.eval(th, to_dev(ev)).cpu().numpy()
    # rates that interference leaves far below their terms are compared to the largest
    assert np.allclose(p, ref, rtol=2e-13, atol=2e-14 * ref.max()), np.max(np.abs(p - ref) / ref)


@pytest.mark.parametrize("near", [True, False])
@pytest.mark.parametrize("reach", REACH)
@pytest.mark.parametrize("w", WIDTHS)
def test_three_body(w, reach, near):
    from paper_1710_08826_amd import Model
    say("wide resolution tddp3", w, reach, near)
    d = mixing(w, reach)
    tau = T.pipipi0_desc()["tau"]
    desc = T.pipipi0_desc(grid=(64, 64), sigma_t=w * tau)
    ev = synth.tddp3_events(N, seed=48)
    ev[2] = times(tau, w * tau, near)
    th = T.truth_theta(x=0.6 * d, y=d)
    v, g = Model(desc).nll(th, to_dev(ev), grad=True)
    vo, go = T.nll_grad(th, ev, desc)
    assert rel_close(v, vo, 1e-12), (v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, r
