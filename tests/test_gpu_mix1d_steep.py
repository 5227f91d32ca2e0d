"""Mixtures with an exponential so steep that its shape spans more than the
exponent range of a double over the observable's range: the other component far
above it and far below it (factors past e^709 both ways), next to every type and
in either order, alone, among three and more; against the oracle, at the tolerances
of the other mixture tests.  The asynchronous call and a batch's first evaluation
give the same values.  Ranges away from zero, an event outside the range.  And
the value of moderately steep ones against extended precision."""
import numpy as np
import pytest
import torch
from scipy.special import erf

from oracle import mix1d as OM
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

PARS = {"gauss": [4.0, 1.3], "exp": [-0.35], "argus": [10.4, -1.7], "bw": [5.5, 0.8]}
LO, HI = 0.0, 10.0


def mixture(types, slopes, lo=LO, hi=HI, shift=0.0):
    """Components of the given types; the exponentials take their slopes in order."""
    comps, th, s = [], [], list(slopes)
    for k, t in enumerate(types):
        comps.append({"type": t, "params": list(range(len(th), len(th) + len(PARS[t])))})
        p = [s.pop(0)] if t == "exp" else [v * (1.0 + 0.11 * k) for v in PARS[t]]
        if t in ("gauss", "bw"):
            p[0] += shift
        th += p
    fr = list(range(len(th), len(th) + len(types) - 1))
    th += [0.37 if len(types) == 2 else 0.9 / len(types)] * len(fr)
    return {"kind": "mix1d", "lo": lo, "hi": hi, "n_params": len(th), "components": comps, "fracs": fr}, np.array(th)


def events(n, seed, lo=LO, hi=HI):
    x = np.random.default_rng(seed).uniform(lo, hi, n)
    # the ends, and a cluster at each: where a steep exponential is not negligible
    x[0], x[-1] = lo + 1e-9 * (hi - lo), hi
    x[1:n // 8] = lo + (hi - lo) * 10.0 ** np.random.default_rng(seed + 1).uniform(-6, -2, n // 8 - 1)
    x[n // 8:n // 4] = hi - (hi - lo) * 10.0 ** np.random.default_rng(seed + 2).uniform(-6, -2, n // 4 - n // 8)
    return x


def compare(d, th, x, tag):
    from paper_1710_08826_amd import Model
    m = Model(d)
    ev = to_dev(x[None])
    v, g = m.nll(th, ev, grad=True)
    vo, go = OM.nll_grad(th, x, d)
    if th.size == 1:  # one exponential: its own closed form (the oracle's quotient rule meets 1/N^2, which underflows)
        D = d["hi"] - d["lo"]
        go = np.array([np.sum(d["lo"] + D / -np.expm1(-th[0] * D) - 1.0 / th[0] - x)])
    assert np.isfinite(vo) and np.isfinite(go).all(), tag
    assert rel_close(v, vo, 1e-12), (tag, v, vo)
    ok, r = grad_close(g, go, 1e-10)
    assert ok, (tag, r)
    assert rel_close(m.nll(th, ev), v, 1e-14)
    out = torch.zeros(1 + m.n_params, device="cuda", dtype=torch.float64)
    m.nll_async(torch.from_numpy(th).cuda(), ev, out)
    o = out.cpu().numpy()
    assert o[0] == v and (o[1:] == g).all(), tag


STEEP = [(("gauss", "exp"), (-80.0,)), (("gauss", "exp"), (-1000.0,)), (("gauss", "exp"), (70.5,)),
         (("exp", "gauss"), (-80.0,)), (("exp", "gauss"), (-1000.0,)), (("exp", "gauss"), (70.5,)),
         (("argus", "exp"), (-80.0,)), (("argus", "exp"), (-1000.0,)), (("exp", "argus"), (-85.0,)),
         (("exp", "argus"), (70.5,)), (("exp", "bw"), (-1000.0,)), (("bw", "exp"), (70.5,)),
         (("exp", "exp"), (-0.35, -80.0)), (("exp", "exp"), (-1000.0, -0.2)), (("exp", "exp"), (70.5, 0.1)),
         (("exp", "exp"), (-80.0, 0.4)), (("exp",), (-60.0,)), (("exp",), (70.5,)),
         (("gauss", "gauss", "exp"), (-80.0,)), (("bw", "exp", "gauss"), (70.5,)),
         (("argus", "bw", "gauss", "exp", "gauss"), (-1000.0,)), (("argus", "bw", "gauss", "exp", "gauss"), (70.5,))]


@pytest.mark.parametrize("types,slopes", STEEP)
def test_steep(types, slopes):
    say("steep mixture", types, slopes)
    d, th = mixture(types, slopes)
    for n in (200, 3000):
        compare(d, th, events(n, 11), (types, slopes, n))


@pytest.mark.parametrize("lo,hi,slope", [(0.0, 1000.0, -0.78), (0.0, 1000.0, -2.0), (5200.0, 5300.0, -0.02),
                                         (5200.0, 5300.0, -0.13), (-1000.0, -900.0, 0.3), (-5.0, 5.0, -130.0)])
def test_ranges(lo, hi, slope):
    """A peak above a background in other ranges (the peak at 0.4 of the range, where it is so wide that no event
    underflows; a factor e^709 lies inside most of them)."""
    say("steep mixture on", lo, hi, slope)
    d, th = mixture(("gauss", "exp"), (slope,), lo, hi)
    th[0], th[1] = lo + 0.4 * (hi - lo), 0.13 * (hi - lo)
    compare(d, th, events(3000, 13, lo, hi), (lo, hi, slope))


@pytest.mark.parametrize("n", [1, 300, 5000])
def test_event_outside_the_range(n):
    """A gentle slope, one event so far outside the range that the broad peak is e^850 above the exponential there."""
    say("mixture, event outside", n)
    d, th = mixture(("gauss", "exp"), (-1.5,))
    th[1] = 60.0
    x = np.random.default_rng(17).uniform(LO, HI, n)
    x[n // 2] = 600.0
    compare(d, th, x, n)


@pytest.mark.parametrize("slope", [-1000.0, -80.0, 70.5])
def test_batch_start(slope):
    from paper_1710_08826_amd import Batch, Model
    say("steep mixture, a batch's start", slope)
    d, th = mixture(("gauss", "exp"), (slope,))
    x = events(3000, 11)
    ev = to_dev(x[None])
    m = Model(d)
    b = Batch(m, 1, 3000)
    b.set([ev], torch.from_numpy(th[None]).cuda())
    b.config(max_iter=1)
    b.run(max_steps=1)
    r = b.results()
    assert r.nll[0] == m.nll(th, ev, grad=True)[0], (r.nll, r.status)
    vo, _ = OM.nll_grad(th, x, d)
    assert rel_close(r.nll[0], vo, 1e-12)


@pytest.mark.parametrize("slope", [-0.35, -4.0, -20.0, -70.0])
def test_value_in_extended_precision(slope):
    """Gaussian and falling exponential, n events: against 80-bit floating point.  Per event the exponent (three
    roundings of an argument that averages 3 where the Gaussian is the density), the exponential's own unit, the
    weights, product and logarithm leave 2e-15 of P, hence n 2e-15 in the sum, whose own roundings are below it;
    with more than one per event in |NLL| that is 2e-15 of it, doubled for the smooth part of the reference."""
    from paper_1710_08826_amd import Model
    say("mixture in extended precision", slope)
    d, th = mixture(("gauss", "exp"), (slope,))
    L = np.longdouble
    for n, seed in ((200, 3), (3000, 4), (40000, 5)):
        x = np.random.default_rng(seed).uniform(LO, HI, n)
        v = Model(d).nll(th, to_dev(x[None]))
        mu, sg, tau, f = (L(t) for t in th)
        xl = x.astype(L)
        N0 = sg * np.sqrt(L(np.pi) / 2) * L(erf((HI - th[0]) / (th[1] * 2 ** 0.5)) - erf((LO - th[0]) / (th[1] * 2 ** 0.5)))
        N1 = np.expm1(tau * L(HI)) / tau
        z = (xl - mu) / sg
        P = f * np.exp(-z * z / 2) / N0 + (1 - f) * np.exp(tau * xl) / N1
        ref = -np.log(P).sum()
        assert abs(ref) > n
        assert abs(L(v) - ref) <= 4e-15 * abs(ref), (n, float(abs(L(v) - ref) / abs(ref)))
