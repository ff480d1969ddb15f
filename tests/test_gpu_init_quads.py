"""Start-pose trials depend on their instance and number alone: a small launch
(a quad of lanes per perspective-3-point trial) gives bit for bit the first
trials of a large one (a lane per trial)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2403_09990_amd import workloads as W

pytestmark = pytest.mark.gpu

LARGE = 400_000  # beyond the quads' range on 256 compute units


@pytest.mark.parametrize("kind,n_kp", [("2d", 6), ("2d", 64), ("3d", 3), ("reg", 3)])
def test_small_launch_gives_the_first_trials_of_a_large_one(kind, n_kp):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng([len(kind), n_kp])
    if kind == "2d":
        inst = W.make_2d3d(rng, n_kp, 2.0, (5.0, 20.0), LARGE)
    elif kind == "3d":
        inst = W.make_3d3d(rng, n_kp, 0.01, 0.05, LARGE)
    else:
        inst = W.make_reg(rng, n_kp, 0.05, 0.01, LARGE)
    ref = P.init(P.DeviceBatch(W.Batch([inst])), P.purse_default_params())
    for m in (1, 15, 16, 17, 65, 4099):
        small = dataclasses.replace(inst, n_samples=m)
        got = P.init(P.DeviceBatch(W.Batch([small])), P.purse_default_params())
        torch.cuda.synchronize()
        assert torch.equal(got["mask"], ref["mask"][:m]), m
        assert torch.equal(got["poses"], ref["poses"][:m]), m
