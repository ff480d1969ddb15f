"""The MEGB's undominated samples on clouds where the rule could go wrong:
bitwise the trace, centre and radii of scanning every sample at every step.

A sample is left out of the shells only if a recent winner is farther by a
margin for every centre of a ball; clouds of equidistant samples, of exact and
of one-ulp copies, of huge and of tiny extent, and around 180 degrees leave
that margin no room, and the sizes cross the shells' capacities (1,280 and
7,168) and the first phase's threshold (32,768).
"""
import numpy as np
import pytest
import torch
from scipy.spatial.transform import Rotation

from paper_2403_09990_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cloud(kind, m, seed):
    """Poses (m, 12): rotations exp(w) R0 and translations with the named spread."""
    rng = np.random.default_rng([seed, m])
    u = rng.normal(size=(2, m, 3))
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    w, t = u
    if kind == "sphere":        # every sample at the radius
        w, t = 0.2 * w, 0.1 * t
    elif kind == "ball":
        w, t = 0.2 * w * rng.random((m, 1)) ** (1 / 3), 0.1 * t * rng.random((m, 1)) ** (1 / 3)
    elif kind == "copies":      # 40 points, each many times
        k = rng.integers(0, 40, m)
        w, t = 0.2 * w[k % m], 0.1 * t[k % m]
    elif kind == "ulps":        # few points, with offsets of the last bits
        k = rng.integers(0, 12, m)
        w = 0.2 * w[k % m] + 1e-7 * rng.normal(size=(m, 3))
        t = 0.1 * t[k % m] + 1e-8 * rng.normal(size=(m, 3))
    elif kind == "wide":        # rotations of every angle
        w, t = np.pi * w * rng.random((m, 1)), 50.0 * t
    elif kind == "tiny":
        w, t = 1e-5 * w, 1e-6 * t
    elif kind == "axis":        # rotations about one axis, points of one line
        a = rng.uniform(-0.5, 0.5, (m, 1))
        w, t = a * np.array([[0.0, 0.0, 1.0]]), a * np.array([[1.0, 2.0, 3.0]])
    else:                       # one sample, m times
        w, t = np.zeros((m, 3)), np.zeros((m, 3))
    R = Rotation.from_rotvec(w).as_matrix() @ Rotation.from_rotvec([0.4, -1.1, 0.7]).as_matrix()
    return np.concatenate([R.reshape(m, 9), t + [0.03, -0.02, 1.0]], 1)


def _check(poses, sizes, megb_iters):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(5)
    db = P.DeviceBatch(W.Batch([W.make_3d3d(rng, 6, 0.01, 0.05, m) for m in sizes]))
    x = torch.as_tensor(poses, dtype=torch.float32, device="cuda").contiguous()
    mask = torch.ones(len(poses), dtype=torch.uint8, device="cuda")
    mask[1::7] = 0              # some infeasible samples among them
    got = []
    for flags in (0, P.PURSE_FLAG_NO_PRUNING):
        status = torch.zeros(len(sizes), dtype=torch.int32, device="cuda")
        got.append(P.megb(db, P.purse_default_params(megb_iters=megb_iters, flags=flags), x, mask, status))
    torch.cuda.synchronize()
    for key in ("trace", "centre", "radii", "n_feasible"):
        assert torch.equal(torch.nan_to_num(got[0][key], 7.0) if got[0][key].is_floating_point() else got[0][key],
                           torch.nan_to_num(got[1][key], 7.0) if got[1][key].is_floating_point() else got[1][key]), key


@pytest.mark.parametrize("kind", ["sphere", "ball", "copies", "ulps", "wide", "tiny", "axis", "one"])
@pytest.mark.parametrize("m", [300, 9001, 40001])
def test_undominated_samples_are_exact(kind, m):
    _check(_cloud(kind, m, 1), [m], 600)


@pytest.mark.parametrize("kind", ["sphere", "ball", "copies", "wide"])
def test_undominated_samples_are_exact_in_shared_compute_units(kind):
    """130 instances: the variant with four chains per compute unit."""
    sizes = [64 + 37 * j for j in range(129)] + [36000]
    _check(np.concatenate([_cloud(kind, m, 2) for m in sizes]), sizes, 300)
