"""Events per workgroup chosen by the sample's size: the values at the sizes
where the choice changes (one event per thread, one round of workgroups filled
exactly and by one event more) against a model with a fixed chunk, which sums
the same terms in another order; and a batch's rows those of the single call."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import grad_close, rel_close, say, to_dev

pytestmark = pytest.mark.gpu


def slots(per_cu):
    return per_cu * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("n", [1, 255, 256, 257, "round", "round+1"])
def test_amplitude_model(n):
    from paper_1710_08826_amd import Model
    d = synth.dalitz_desc(grid=(64, 64))
    n = {"round": 256 * slots(2), "round+1": 256 * slots(2) + 1}.get(n, n)
    say("chunk rule dalitz n =", n)
    ev = to_dev(synth.dalitz_events(n, seed=81))
    th = synth.dalitz_truth() * 1.01
    v, g = Model(d).nll(th, ev, grad=True)
    vo, go = Model(dict(d, chunk=4096)).nll(th, ev, grad=True)
    # the same per-event terms, summed in another order: a few units over up to 1e5 terms
    assert rel_close(v, vo, 1e-13), (v, vo)
    ok, r = grad_close(g, go, 1e-12)
    assert ok, r


@pytest.mark.parametrize("extra", [0, 1])
def test_mixture_and_batch(extra):
    from paper_1710_08826_amd import Batch, Model
    n = 1024 * slots(8) + extra
    say("chunk rule mix n =", n)
    m = Model(synth.mix1d_desc())
    th = synth.mix1d_truth()
    g = torch.Generator(device="cuda").manual_seed(3)
    ev = (torch.rand((1, n), generator=g, device="cuda", dtype=torch.float64) - 0.5) * 18.0
    v, gr = m.nll(th, ev, grad=True)
    vo, go = Model(dict(synth.mix1d_desc(), chunk=1024)).nll(th, ev, grad=True)
    assert rel_close(v, vo, 1e-13), (v, vo)
    ok, r = grad_close(gr, go, 1e-12)
    assert ok, r
    # the batch takes the same rows: its first evaluation is the single one's bits
    b = Batch(m, 2, n)
    small = ev[:, :3000].contiguous()
    b.set([ev, small], torch.from_numpy(np.stack([th, th])).cuda())
    b.config(max_iter=0)
    b.step()
    torch.cuda.synchronize()
    _, _, nll, _ = b.status()
    assert np.isfinite(nll).all()
    b2 = Batch(m, 1, n)
    b2.set([ev], torch.from_numpy(th[None]).cuda())
    b2.run()
    b.config(max_iter=500)
    b.set([ev, small], torch.from_numpy(np.stack([th, th])).cuda())
    b.run()
    assert b.results().nll[0] == b2.results().nll[0]
    assert b2.results().nll[0] == m.nll(b2.results().theta[0], ev, grad=True)[0]
