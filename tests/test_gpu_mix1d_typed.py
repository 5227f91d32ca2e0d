"""The passes compiled per component types (one or two components, in every
order): value and gradient against the oracle at sizes around the groups of
four events per thread and the chunk; a pivot exponential at the end of the
range where its factor is small; events on the edges of the range."""
import numpy as np
import pytest

from oracle import mix1d as OM
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

PARS = {"gauss": [4.0, 1.3], "exp": [-0.35], "argus": [10.4, -1.7], "bw": [5.5, 0.8]}
TYPES = sorted(PARS)
LO, HI = 0.0, 10.0


def model(types):
    comps, th = [], []
    for k, t in enumerate(types):
        comps.append({"type": t, "params": list(range(len(th), len(th) + len(PARS[t])))})
        th += [v * (1.0 + 0.11 * k) for v in PARS[t]]
    fr = [len(th)] if len(types) == 2 else []
    th += [0.37] * len(fr)
    return {"kind": "mix1d", "lo": LO, "hi": HI, "n_params": len(th), "components": comps, "fracs": fr}, np.array(th)


def compare(d, th, x, tag):
    from paper_1710_08826_amd import Model
    m = Model(d)
    v, g = m.nll(th, to_dev(x[None]), grad=True)
    vo, go = OM.nll_grad(th, x, d)
    assert rel_close(v, vo, 1e-12), (tag, v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, (tag, r)
    assert rel_close(m.nll(th, to_dev(x[None])), v, 1e-14)


@pytest.mark.parametrize("types", [(a,) for a in TYPES] + [(a, b) for a in TYPES for b in TYPES])
def test_signatures(types):
    d, th = model(types)
    for n in (1, 255, 1023, 1024, 1025, 4096 + 1024 + 7):
        say("typed mixture", types, n)
        x = np.random.default_rng(n).uniform(LO + 1e-3, HI - 1e-3, n)
        x[0] = LO + 1e-6
        x[-1] = HI
        compare(d, th, x, (types, n))


@pytest.mark.parametrize("tau", [-20.0, 0.0, 12.0])
def test_steep_pivot(tau):
    """Factors of the pivot from e^-200 to 1 (and its flat limit)."""
    d, th = model(("gauss", "exp"))
    th[2] = tau
    say("steep pivot", tau)
    x = np.random.default_rng(2).uniform(LO, HI, 3000)
    compare(d, th, x, tau)
