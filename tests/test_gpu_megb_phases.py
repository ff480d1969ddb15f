"""The descent's phases at their edges, bitwise against scanning every sample at
every step: descents that end within the first phase, at its end and shortly
after it, on sizes on either side of the lines that set its length (32,768;
65,536; 2^17; 2^19 samples, and with four chains a compute unit 65,536 and
2^19), on clouds whose undominated samples overflow their slots, leave their
ball, or rule nothing out.  And the exact ball where the search over the
undominated samples has to start again over every sample."""
import numpy as np
import pytest
import torch

from paper_2403_09990_amd import workloads as W
from tests.test_gpu_megb_domination import _check, _cloud

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ball", "sphere", "wide"])
@pytest.mark.parametrize("m", [9001, 33000, 65535, 131073, 530001])
def test_short_descents(kind, m):
    cloud = _cloud(kind, m, 4)
    for iters in (10, 11, 26, 27, 28, 36, 43, 60, 80):
        print(kind, m, iters, flush=True)
        _check(cloud, [m], iters)


@pytest.mark.parametrize("kind", ["ball", "sphere"])
def test_short_descents_in_shared_compute_units(kind):
    sizes = [700 + 41 * j for j in range(126)] + [33001, 65537, 140001, 530001]
    cloud = np.concatenate([_cloud(kind, m, 6) for m in sizes])
    for iters in (12, 42, 43, 80):
        print(kind, iters, flush=True)
        _check(cloud, sizes, iters)


@pytest.mark.parametrize("kind", ["flat", "ball"])
def test_exact_ball_of_an_early_centre(kind):
    """30 steps leave the descent's centre far from the exact one: outside the
    ball the undominated samples hold for.  The radii about the exact centre
    (rounded to float32, 6e-8 of a distance of one about radii of 0.1) agree with
    those of a search without them to 2e-6."""
    import paper_2403_09990_amd as P
    m = 70001
    cloud = _cloud("ball", m, 8)
    if kind == "flat":  # (translations in a thin plate: the descent zigzags)
        cloud[:, 9:] = [0.03, -0.02, 1.0] + (cloud[:, 9:] - [0.03, -0.02, 1.0]) * [1.0, 0.3, 0.001]
    db = P.DeviceBatch(W.Batch([W.make_3d3d(np.random.default_rng(5), 6, 0.01, 0.05, m)]))
    x = torch.as_tensor(cloud, dtype=torch.float32, device="cuda").contiguous()
    mask = torch.ones(m, dtype=torch.uint8, device="cuda")
    radii = []
    for flags in (P.PURSE_FLAG_EXACT_MEB, P.PURSE_FLAG_EXACT_MEB | P.PURSE_FLAG_NO_PRUNING):
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        gp = P.purse_default_params(megb_iters=30, megb_avg=3, flags=flags)
        radii.append(P.megb(db, gp, x, mask, status)["radii"].cpu().numpy())
    assert np.allclose(radii[0], radii[1], rtol=2e-6, atol=0.0)
