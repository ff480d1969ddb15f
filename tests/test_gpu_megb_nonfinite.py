"""Balls of clouds that hold a sample which is no number (purse_megb takes the
poses and masks of any program): the call ends, in the shells' steps as in the
scans, and the component without such a sample is bitwise that of the clean
cloud.  Sizes on either side of the shells' capacity and of the first phase's
threshold."""
import numpy as np
import pytest
import torch

from paper_2403_09990_amd import workloads as W
from tests.test_gpu_megb_domination import _cloud

pytestmark = pytest.mark.gpu

FLAGS = ("PURSE_FLAG_NO_PRUNING", "PURSE_FLAG_EXACT_MEB")


def _ball(P, poses, flags):
    db = P.DeviceBatch(W.Batch([W.make_3d3d(np.random.default_rng(5), 6, 0.01, 0.05, len(poses))]))
    x = torch.as_tensor(poses, dtype=torch.float32, device="cuda").contiguous()
    mask = torch.ones(len(poses), dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = P.megb(db, P.purse_default_params(megb_iters=300, flags=flags), x, mask, status)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("m", [300, 9001, 40001])
@pytest.mark.parametrize("flag", [None, *FLAGS])
@pytest.mark.parametrize("part,sample,value", [("t", 0, np.nan), ("t", 57, np.nan), ("t", 57, np.inf),
                                               ("t", 57, 3e19), ("R", 0, np.nan), ("R", 57, np.inf)])
def test_samples_that_are_no_numbers(m, flag, part, sample, value):
    import paper_2403_09990_amd as P
    flags = 0 if flag is None else getattr(P, flag)
    clean = _cloud("ball", m, 3)
    poses = clean.copy()
    poses[sample, 9 if part == "t" else 4] = value
    print(m, flag, part, sample, value, flush=True)
    got, ref = _ball(P, poses, flags), _ball(P, clean, flags)
    assert got["n_feasible"][0] == m
    c = 0 if part == "t" else 1  # the other component's chain
    assert np.array_equal(got["trace"][..., c], ref["trace"][..., c])
    own = slice(0, 9) if c == 0 else slice(9, 12)
    assert np.array_equal(got["centre"][:, own], ref["centre"][:, own])
    assert got["radii"][0, c] == ref["radii"][0, c]
