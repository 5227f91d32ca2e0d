"""Batch steps at the edges of their launches: 1, 64, 65 and 130 fits (tables of
64 fits per workgroup, a search of 64 entries per round), mixtures of two, four
and nine parameters (the minimizer's register copies and the general form),
step counts that don't fill a graph.  A fit ends where it ends alone, bit for
bit, and its NLL is the single-fit one at its parameters."""
import numpy as np
import pytest

from tests.gpu_util import rel_close, say, to_dev

pytestmark = pytest.mark.gpu

LO, HI = 0.0, 10.0
MIXTURES = {
    2: ([("gauss", [4.0, 1.3])], []),
    4: ([("gauss", [4.0, 0.7]), ("exp", [-0.35])], [0.4]),
    9: ([("gauss", [3.0, 0.4]), ("gauss", [7.0, 0.5]), ("bw", [5.0, 0.3]), ("exp", [-0.2])], [0.3, 0.3]),
}


def mixture(P):
    comps, fr = MIXTURES[P]
    th, out = [], []
    for t, p in comps:
        out.append({"type": t, "params": list(range(len(th), len(th) + len(p)))})
        th += p
    if P == 9:  # the first two fractions free, the third shares the second's parameter
        f = [len(th), len(th) + 1, len(th) + 1]
    else:
        f = list(range(len(th), len(th) + len(fr)))
    th += fr
    return {"kind": "mix1d", "lo": LO, "hi": HI, "n_params": len(th), "components": out, "fracs": f}, np.array(th)


def events(P, n, seed):
    rng = np.random.default_rng(1000 * P + seed)
    x = rng.uniform(LO, HI, n)
    k = rng.random(n)
    x = np.where(k < 0.35, rng.normal(4.0, 0.7, n), x)
    x = np.where(k > 0.7, rng.exponential(3.0, n), x)
    return np.clip(x, LO, HI)


@pytest.mark.parametrize("P", sorted(MIXTURES))
def test_steps(P):
    from paper_1710_08826_amd import Batch, Model
    d, th = mixture(P)
    m = Model(d)
    evs = [to_dev(events(P, 200 + (37 * i * i) % 2900, i)[None]) for i in range(130)]
    alone = {}
    for F in (1, 64, 65, 130):
        say("batch steps", P, F)
        b = Batch(m, F, 3200)
        for i in range(F):
            b.set_slot(i, evs[i], th * (1.0 + 0.02 * np.sin(i + np.arange(th.size))))
        b.run(13, 5)  # five, five and three
        b.run(3, 3)
        _, running = b.run(2000, 9)
        assert running == 0
        r = b.results()
        for i in sorted({0, 1, F // 2, F - 1} & set(range(F))):
            assert r.status[i] in (2, 3)
            assert rel_close(m.nll(r.theta[i], evs[i]), r.nll[i], 1e-13)
            key = (r.status[i], r.theta[i].tobytes(), r.nll[i], r.errors[i].tobytes(), r.iters[i], r.n_evals[i])
            if i not in alone:
                one = Batch(m, 1, 3200)
                one.set_slot(0, evs[i], th * (1.0 + 0.02 * np.sin(i + np.arange(th.size))))
                one.run(2000, 8)
                q = one.results()
                alone[i] = (q.status[0], q.theta[0].tobytes(), q.nll[0], q.errors[0].tobytes(), q.iters[0], q.n_evals[0])
            assert key == alone[i], (P, F, i)
