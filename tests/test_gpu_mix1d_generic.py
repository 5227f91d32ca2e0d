"""The passes of mixtures of three to eight components (types at run time, four
or eight held): value and gradient against the oracle at sizes around the two
events per thread and round and the chunk, shared parameters, an Argus end point
inside the range."""
import numpy as np
import pytest

from oracle import mix1d as OM
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

PARS = {"gauss": [4.0, 1.3], "exp": [-0.35], "argus": [9.4, -1.7], "bw": [5.5, 0.8]}
MIXES = [("gauss", "gauss", "exp"), ("exp", "argus", "bw"), ("bw", "exp", "gauss", "argus"),
         ("argus", "bw", "gauss", "exp", "gauss"), ("gauss", "exp", "bw", "argus", "gauss", "exp", "bw", "gauss")]
LO, HI = 0.0, 10.0


def mixture(types):
    comps, th = [], []
    for k, t in enumerate(types):
        if k and t == "gauss" and types[0] == "gauss":  # the first Gaussian's mean, its own width
            comps.append({"type": t, "params": [0, len(th)]})
            th.append(0.4 + 0.3 * k)
            continue
        comps.append({"type": t, "params": list(range(len(th), len(th) + len(PARS[t])))})
        th += [v * (1.0 + 0.07 * k) for v in PARS[t]]
    fr = list(range(len(th), len(th) + len(types) - 1))
    th += [0.9 / len(types)] * len(fr)
    return {"kind": "mix1d", "lo": LO, "hi": HI, "n_params": len(th), "components": comps, "fracs": fr}, np.array(th)


@pytest.mark.parametrize("types", MIXES)
def test_generic(types):
    from paper_1710_08826_amd import Model
    d, th = mixture(types)
    m = Model(d)
    for n in (1, 255, 256, 257, 511, 513, 1024, 1025, 4096 + 700):
        say("generic mixture", types, n)
        x = np.random.default_rng(n).uniform(LO + 1e-3, HI, n)
        v, g = m.nll(th, to_dev(x[None]), grad=True)
        vo, go = OM.nll_grad(th, x, d)
        assert rel_close(v, vo, 1e-12), (n, v, vo)
        ok, r = grad_close(g, go, 1e-10)
        assert ok, (n, r)
        assert rel_close(m.nll(th, to_dev(x[None])), v, 1e-14)
