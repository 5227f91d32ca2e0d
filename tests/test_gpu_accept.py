"""Accept-reject generation by waves: the same events whatever the number of
events per wave and of lanes per event (runs of every size are prefixes of a
large one, bit for bit), and the limits: no event resolved, none above or all
above the envelope."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 255, 4096, 4097, 12_289, 70_001]


@pytest.mark.parametrize("kind", ["dalitz3", "tddp3", "td4"])
def test_prefixes(kind):
    from paper_1710_08826_amd import Model
    big = {"dalitz3": 540_000, "tddp3": 300_000, "td4": 20_000}[kind]
    d, th = {"dalitz3": (synth.dalitz_desc(grid=(256, 256)), synth.dalitz_truth()),
             "tddp3": (synth.tddp3_desc(grid=(256, 256)), synth.tddp3_truth()),
             "td4": (synth.td4_desc(), synth.td4_truth())}[kind]
    m = Model(d)
    if kind == "td4":
        m.generate_norm_sample(2_000_000, 7)
    ev, W = m.generate(th, big, seed=21)
    W *= 1.5
    ev, _ = m.generate(th, big, seed=21, envelope=W)
    assert bool(torch.isfinite(ev).all())
    for n in [s for s in SIZES if s <= big]:
        say("accept prefix", kind, n)
        part, _ = m.generate(th, n, seed=21, envelope=W)
        assert torch.equal(part, ev[:, :n])


@pytest.mark.parametrize("n", [1, 70])
def test_limits(n):
    from paper_1710_08826_amd import FitNLLError, Model
    m = Model(synth.dalitz_desc(grid=(64, 64)))
    th = synth.dalitz_truth()
    say("accept limits", n)
    with pytest.raises(FitNLLError, match=f"{n} events not resolved"):
        m.generate(th, n, seed=3, envelope=1e30)
    with pytest.raises(FitNLLError, match=f"{n} accepted events lie above"):
        m.generate(th, n, seed=3, envelope=1e-30)
    bad = np.zeros_like(th)
    with pytest.raises(FitNLLError, match="vanishes"):
        m.generate(bad, n, seed=3)
