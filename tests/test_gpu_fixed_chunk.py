"""Events passes whose threads take several events each: a fixed chunk of 1024,
2048 or 4096 events per workgroup at one event less and more than whole
workgroups, and at a last one with a full and a partial round, for every
amplitude model, structure, gradient level and number of events per thread;
against the oracle (twenty four-body amplitudes: against one event per thread).
Without a fixed chunk samples below 131072 events get one event per thread,
which leaves the loads ahead and the second round untested at the sizes an
oracle takes.  Tolerances are those of the models' own tests."""
import numpy as np
import pytest

import synth
from oracle import dalitz3 as OD, td4 as OT, tddp3 as T
from tests.gpu_util import grad_close, rel_close, say, to_dev
from tests.test_gpu_shapes import DALITZ_SHAPES
from tests.test_gpu_tddp3_shared import TABLES

pytestmark = pytest.mark.gpu

CHUNKS = [1024, 2048, 4096]


def sizes(chunk):
    return [chunk - 1, 2 * chunk + 1, 2 * chunk + 257]


def compare(m, th, ev, oracle, gtol, tag):
    v, g = m.nll(th, to_dev(ev), grad=True)
    vo, go = oracle(th, ev)
    assert rel_close(v, vo, 1e-12), (tag, v, vo)
    ok, r = grad_close(g, go, gtol)
    assert ok, (tag, r.max())
    assert rel_close(m.nll(th, to_dev(ev)), v, 1e-14), tag


@pytest.mark.parametrize("chunk", CHUNKS)
@pytest.mark.parametrize("ept", [1, 2])
@pytest.mark.parametrize("free", [False, True])
def test_dalitz(free, ept, chunk):
    from paper_1710_08826_amd import Model
    d = synth.dalitz_desc(grid=(64, 64), free_lineshapes=free)
    th0 = synth.dalitz_truth(free_lineshapes=free)
    th = th0 * (1.0 + 0.01 * np.cos(np.arange(th0.size)))
    m = Model(dict(d, chunk=chunk, events_per_thread=ept))
    cells = OD.Dalitz(d).grid_cells()
    for n in sizes(chunk):
        say("fixed chunk dalitz", free, ept, chunk, n)
        compare(m, th, synth.dalitz_events(n, seed=n), lambda t, e: OD.nll_grad(t, e, d, cells), 1e-9, (free, ept, n))


@pytest.mark.parametrize("free", [False, True])
@pytest.mark.parametrize("name", ["one_pair_L0_L2", "spin2_all_pairs"])
def test_dalitz_structures(name, free):
    from paper_1710_08826_amd import Model
    res = DALITZ_SHAPES[name]
    d = OD.config1_desc(grid=(64, 64), free_lineshapes=free, resonances=res)
    th = OD.truth_theta(d, resonances=res) * (1.0 + 0.02 * np.cos(np.arange(2 * len(res) * (2 if free else 1))))
    cells = OD.Dalitz(d).grid_cells()
    for ept in (1, 2):
        m = Model(dict(d, chunk=1024, events_per_thread=ept))
        for n in sizes(1024):
            say("fixed chunk dalitz shape", name, free, ept, n)
            compare(m, th, synth.dalitz_events(n, seed=n), lambda t, e: OD.nll_grad(t, e, d, cells), 1e-9, (name, ept, n))


@pytest.mark.parametrize("chunk", CHUNKS)
@pytest.mark.parametrize("wide", [False, True])
def test_mixing_three_body(wide, chunk):
    from paper_1710_08826_amd import Model
    d = (synth.tddp3_desc16 if wide else synth.tddp3_desc)(grid=(64, 64))
    th = (synth.tddp3_truth16 if wide else synth.tddp3_truth)()
    th = th * (1.0 + 0.01 * np.cos(np.arange(th.size)))
    m = Model(dict(d, chunk=chunk))
    for n in sizes(chunk):
        say("fixed chunk tddp3", wide, chunk, n)
        compare(m, th, synth.tddp3_events(n, seed=n), lambda t, e: T.nll_grad(t, e, d), 1e-10, (wide, n))


@pytest.mark.parametrize("name", sorted(TABLES))
def test_mixing_three_body_structures(name):
    from paper_1710_08826_amd import Model
    res = TABLES[name]
    d = T.pipipi0_desc(grid=(64, 64), resonances=res)
    th = T.truth_theta(resonances=res, x=0.02, y=0.03)
    k = 2 * len(res)
    th[k:2 * k] = th[k:2 * k] * 0.9 + 0.05
    m = Model(dict(d, chunk=1024))
    for n in sizes(1024):
        say("fixed chunk tddp3 shape", name, n)
        compare(m, th, synth.tddp3_events(n, seed=n), lambda t, e: T.nll_grad(t, e, d), 1e-10, (name, n))


@pytest.mark.parametrize("chunk", CHUNKS)
def test_four_body(chunk):
    from paper_1710_08826_amd import Model
    d, th = synth.td4_desc(), synth.td4_truth()
    th = th * (1.0 + 0.01 * np.cos(np.arange(th.size)))
    mc = synth.td4_phase_space(2000, seed=41)
    m = Model(dict(d, chunk=chunk))
    m.set_norm_sample(to_dev(mc))
    for n in sizes(chunk):
        say("fixed chunk td4", chunk, n)
        compare(m, th, synth.td4_events(n, seed=n), lambda t, e: OT.nll_grad(t, e, mc, d), 1e-10, n)


@pytest.mark.parametrize("chunk", CHUNKS)
def test_four_body_split(chunk):
    """Twenty amplitudes, whose gradients events at interference minima keep the oracle from resolving: against one
    event per thread, which sums the same per-event terms in another order."""
    from paper_1710_08826_amd import Model
    d, th = synth.td4_split_desc(), synth.td4_split_truth()
    th = th * (1.0 + 0.01 * np.cos(np.arange(th.size)))
    mc = to_dev(synth.td4_phase_space(2000, seed=41))
    m, one = Model(dict(d, chunk=chunk)), Model(dict(d, chunk=256))
    m.set_norm_sample(mc)
    one.set_norm_sample(mc)
    for n in sizes(chunk):
        say("fixed chunk td4 split", chunk, n)
        ev = to_dev(synth.td4_events(n, seed=n))
        (v, g), (vo, go) = m.nll(th, ev, grad=True), one.nll(th, ev, grad=True)
        # as in the tests of the rule: a few units over up to 1e5 terms
        assert rel_close(v, vo, 1e-13), (n, v, vo)
        ok, r = grad_close(g, go, 1e-12)
        assert ok, (n, r)


@pytest.mark.parametrize("amps", [[[0, 0, 0], [0, 1, 1], [0, 2, 0]], [[0, 0, 4], [0, 0, 5], [0, 0, 3]]])
def test_four_body_structures(amps):
    from paper_1710_08826_amd import Model
    spin1 = amps[0][2] == 4
    d = synth.td4_desc(r12=((1, 1.019461, 0.004249),), r34=((1, 0.77526, 0.1491),)) if spin1 else \
        synth.td4_desc(r12=((0, 0.0, 0.0),))
    d["amps"] = amps
    th = np.array([0.3, 0.1, -0.2, 0.25, 0.15, -0.05, 1.0, 0.0, 0.6, -0.4, 0.3, 0.2, 0.05, -0.03])
    mc = synth.td4_phase_space(2000, seed=74)
    m = Model(dict(d, chunk=1024))
    m.set_norm_sample(to_dev(mc))
    for n in sizes(1024):
        say("fixed chunk td4 shape", spin1, n)
        compare(m, th, synth.td4_events(n, seed=n), lambda t, e: OT.nll_grad(t, e, mc, d), 1e-10, (spin1, n))


@pytest.mark.parametrize("kind", ["dalitz3 free", "tddp3", "td4"])
def test_presummed_rows(kind):
    """Row sets long enough to be pre-summed by their own workgroups (above 256 KB, which the rule's rows reach only
    for the widest rows), the last of them short: against few rows, which are not."""
    from paper_1710_08826_amd import Model
    n = 300 * 1024 + 300
    say("presummed rows", kind)
    if kind == "dalitz3 free":
        d, th = synth.dalitz_desc(grid=(256, 256), free_lineshapes=True), synth.dalitz_truth(free_lineshapes=True)
        ev = synth.dalitz_events(n, seed=5)
    elif kind == "tddp3":
        d, th, ev = synth.tddp3_desc16(grid=(64, 64)), synth.tddp3_truth16(), synth.tddp3_events(n, seed=5)
    else:
        d, th, ev = synth.td4_split_desc(), synth.td4_split_truth(), synth.td4_events(n, seed=5)
    many, few = Model(dict(d, chunk=256)), Model(dict(d, chunk=16384))
    if kind == "td4":
        mc = to_dev(synth.td4_phase_space(2000, seed=41))
        many.set_norm_sample(mc)
        few.set_norm_sample(mc)
    th = th * (1.0 + 0.01 * np.cos(np.arange(th.size)))
    ev = to_dev(ev)
    (v, g), (vo, go) = many.nll(th, ev, grad=True), few.nll(th, ev, grad=True)
    # as in the tests of the rule: a few units over up to 1e5 terms
    assert rel_close(v, vo, 1e-13), (v, vo)
    ok, r = grad_close(g, go, 1e-12)
    assert ok, r
