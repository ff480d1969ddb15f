"""An instance's gradients are bitwise the same in every batch: alone, among
four, five and seventy (a call of few instances must not take other arithmetic
than one of many), with the passes' tape short and at its longest."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import _grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_inst,iters", [(4, 30), (5, 30), (70, 30), (5, 134)])
def test_gradients_do_not_depend_on_the_batch(n_inst, iters):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng([n_inst, iters])
    insts = [W.make_2d3d(rng, int(rng.integers(6, 49)), 2.0, (5.0, 20.0), 300) if j % 2 == 0 else
             W.make_3d3d(rng, int(rng.integers(6, 49)), 0.01, 0.05, 300) for j in range(n_inst)]
    gp = P.purse_default_params(n_iters=iters, megb_iters=600)
    g_radii, g_centre = rng.normal(size=(n_inst, 2)), rng.normal(size=(n_inst, 6))
    res = PT.run_gpu(W.Batch(insts), gp)
    got, status = _grads(P, res, gp, 0, g_radii, g_centre)
    assert (status & 0xFF == P.PURSE_BWD_OK).all()
    ko = res["db"].kp_off_host
    for j in (0, 1, n_inst - 2, n_inst - 1):
        one = PT.run_gpu(W.Batch([insts[j]]), gp)
        alone, _ = _grads(P, one, gp, 0, g_radii[j:j + 1], g_centre[j:j + 1])
        for a, c in zip(got, alone):
            assert np.array_equal(a[ko[j]:ko[j + 1]], c), j
