"""Normalization matrices on the matrix cores: numbers of amplitudes that leave
the 16 x 16 tiles full, nearly empty or split, numbers of points around a
wave's 64, a workgroup's 256 and one round of workgroups, grids with waves
inside, outside and across the region; normalization and its gradient against
the oracle (tolerances of the models' own normalization tests)."""
import numpy as np
import pytest
import torch

import synth
from oracle import common, dalitz3 as D, td4 as OT, tddp3 as T
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu

AMPS = synth.td4_split_desc()["amps"]


def td4_case(k):
    d = synth.td4_split_desc()
    d["amps"] = [a[:3] + [("A", "Abar", "both")[(i + k) % 3]] for i, a in enumerate(AMPS[:k])]
    d["amps"][0][3] = "both"
    n = sum({"both": 2}.get(a[3], 1) for a in d["amps"])
    th = np.concatenate([np.sin(np.arange(2 * n) + 1.0), [0.02, -0.03]])
    return d, th


@pytest.mark.parametrize("k,points", [(1, 1), (2, 63), (8, 64), (9, 65), (16, 257), (17, 700), (20, 512 * 256 + 1)])
def test_four_body(k, points):
    from paper_1710_08826_amd import Model
    say("gram td4 K =", k, "points =", points)
    d, th = td4_case(k)
    mc = synth.td4_phase_space(points, seed=52)
    m = Model(d)
    m.set_norm_sample(to_dev(mc))
    I, dI = m.norm(th)
    t = torch.tensor(th, requires_grad=True)
    ir = OT.TD4(d).integrated_rate(t, torch.tensor(mc))
    ir.mean().backward()
    assert rel_close(I, common.fsum(ir.detach()) / points, 1e-12)
    ok, r = grad_close(dI, t.grad.numpy(), 1e-11)
    assert ok, r


@pytest.mark.parametrize("k", [1, 7, 8])
@pytest.mark.parametrize("grid", [(2, 3), (5, 300), (257, 129)])
def test_three_body(k, grid):
    from paper_1710_08826_amd import Model
    say("gram dalitz K =", k, grid)
    d = synth.dalitz_desc(grid=grid)
    d["resonances"] = d["resonances"][:k]
    th = synth.dalitz_truth()[:2 * k]
    I, dI = Model(d).norm(th)
    model = D.Dalitz(d)
    t = torch.tensor(th, requires_grad=True)
    nt = D.norm_tensor(model, t)
    nt.backward()
    assert rel_close(I, D.norm_value(model, th), 1e-12)
    ok, r = grad_close(dI, t.grad.numpy(), 1e-11)
    assert ok, r


@pytest.mark.parametrize("k,grid", [(1, (40, 40)), (5, (33, 33)), (16, (130, 130))])
def test_mixing_three_body(k, grid):
    from paper_1710_08826_amd import Model
    say("gram tddp3 K =", k, grid)
    res = synth.TDDP_RESONANCES16[:k]
    d = synth.tddp3_desc(grid=grid, resonances=res)
    th = synth.tddp3_truth(x=0.1, y=-0.2, resonances=res)
    th[2 * k:4 * k] = 0.8 * th[2 * k:4 * k] + 0.07
    I, dI = Model(d).norm(th)
    t = torch.tensor(th, requires_grad=True)
    nt = T.norm_tensor(T.TDDP(d), t)
    nt.backward()
    assert rel_close(I, T.norm_value(T.TDDP(d), th), 1e-12)
    ok, r = grad_close(dI, t.grad.numpy(), 1e-11)
    assert ok, r
