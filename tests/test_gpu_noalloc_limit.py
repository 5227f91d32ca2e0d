"""The allocation-free call at its scratch array's limit, on a model whose
normalization matrix is not built yet: samples whose partial rows leave only a
few hundred doubles of it free are taken, with the results of fn_nll_async."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

CAP = 1 << 21  # doubles of the scratch array (fitnll.h)


def sample(ev, n):
    """n events, repeating the columns of ev (leading dimension n)."""
    return to_dev(ev).repeat(1, -(-n // ev.shape[1]))[:, :n].contiguous()


@pytest.mark.parametrize("kind", ["dalitz3", "tddp3"])
def test_first_call_at_the_limit(kind):
    from paper_1710_08826_amd import FitNLLError, Model
    if kind == "tddp3":
        d, th = synth.tddp3_desc16(grid=(64, 64)), synth.tddp3_truth16()
        ev = synth.tddp3_events(100_000, seed=44)
    else:
        d, th = synth.dalitz_desc(grid=(64, 64)), synth.dalitz_truth()
        ev = synth.dalitz_events(100_000, seed=44)
    d["chunk"] = 256
    nv = th.size + 1
    rows = next(r for r in range(CAP // nv, 0, -1) if (r + -(-r // 16)) * nv <= CAP - 512)
    n = 256 * rows
    say("noalloc limit", kind, rows, "rows,", n, "events")
    evd = sample(ev, n)
    tdev = torch.from_numpy(th).cuda()
    out = torch.zeros(2, nv, device="cuda", dtype=torch.float64)
    fresh, ref = Model(d), Model(d)
    fresh.nll_async_noalloc(tdev, evd, out[0])
    ref.nll_async(tdev, evd, out[1])
    assert torch.isfinite(out[1]).all() and torch.equal(out[0], out[1])
    # the cached matrix is whole: another sample, and the array's own limit
    fresh.nll_async_noalloc(tdev, evd[:, :5000], out[0])
    ref.nll_async(tdev, evd[:, :5000], out[1])
    assert torch.equal(out[0], out[1])
    over = sample(ev, n + 256 * 64)
    with pytest.raises(FitNLLError, match="scratch"):
        Model(d).nll_async_noalloc(tdev, over, out[0])
