"""The random walk against the oracle where its lanes and rounds run out: two,
a full and a partial last slot of perturbations, one kept perturbation and the
most, one scale and the most, odd and even keypoint counts."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests.test_gpu_walk import _compare, _run, _starts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_kp,n_perturb,n_keep,n_scales",
                         [(6, 2, 1, 1), (7, 64, 16, 32), (13, 65, 3, 15), (8, 256, 16, 4), (9, 150, 7, 31)])
@pytest.mark.parametrize("kind", ["2d", "3d"])
def test_walk_edges_match_oracle(kind, n_kp, n_perturb, n_keep, n_scales):
    rng = np.random.default_rng([n_kp, n_perturb])
    if kind == "2d":
        inst = W.make_2d3d(rng, n_kp, 2.0, (5.0, 20.0), 64)
        kw = dict(omega0=0.5, v0=0.05, t_pert=0.005, r_pert=0.02)
    else:
        inst = W.make_3d3d(rng, n_kp, 0.01, 0.05, 64)
        kw = dict(omega0=0.3, v0=0.05, t_pert=0.01, r_pert=0.05)
    starts = _starts(inst, 8, 20)
    assert len(starts) > 0
    kw.update(n_walks=2, n_iters=4, n_perturb=n_perturb, n_keep=n_keep, n_scales=n_scales)
    db, gp, wp, off, res = _run(W.Batch([inst]), [starts], kw)
    st = _compare(inst, starts, res, 0, off, gp, wp)
    assert st["same"] > 0
