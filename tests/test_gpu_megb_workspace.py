"""A workspace of the size asked for before the undominated samples' slots grew
(one slot for 16 samples instead of 8, and a larger first-phase scratch) still
serves the sampler, the ball and its gradient, with the same results."""
import numpy as np
import pytest
import torch

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import _grads

pytestmark = pytest.mark.gpu


def _align(x):
    return (x + 255) // 256 * 256


def _slots(total, div):
    return _align(4 * 2 * (total // div + 1)) + _align(16 * 2 * (total // div + 1))


@pytest.mark.parametrize("sizes", [[40000], [33333, 70001, 12]])
def test_earlier_workspace_size(sizes):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(sizes)
    b = W.Batch([W.make_3d3d(rng, 8, 0.01, 0.05, m) for m in sizes])
    gp = P.purse_default_params(n_iters=10, megb_iters=600)
    res = PT.run_gpu(b, gp)
    db, n = res["db"], len(sizes)
    now = P.purse_workspace_size(db, gp)
    rest = now - _slots(sum(sizes), 8)         # up to the slots, with today's first-phase scratch
    earlier = rest + _slots(sum(sizes), 16)    # (that scratch was larger, so this is at most the earlier size)
    assert earlier < now
    ws = torch.empty(earlier, dtype=torch.uint8, device="cuda")
    out = P.sample(db, gp, ws=ws)
    small = P.megb(db, gp, out["poses"], out["mask"], out["inst_status"], ws=ws)
    for key in ("trace", "centre", "radii"):
        assert torch.equal(res[key], small[key]), key
    g_radii, g_centre = rng.normal(size=(n, 2)), rng.normal(size=(n, 6))
    want, _ = _grads(P, res, gp, 0, g_radii, g_centre)
    got, _ = _grads(P, dict(res, ws=ws), gp, 0, g_radii, g_centre)
    for a, c in zip(want, got):
        assert np.array_equal(a, c)
    with pytest.raises(P.PurseError):
        P.megb(db, gp, out["poses"], out["mask"], out["inst_status"], ws=ws[:earlier - 1])
