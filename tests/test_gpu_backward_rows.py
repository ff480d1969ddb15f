"""The 3D-3D reverse sweep against the oracle on either side of the rows that
keep the targets' matrices (91 iterations, not 92), alone and in a batch."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import RTOL, _grads, _oracle, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_inst,iters", [(1, 91), (1, 92), (6, 91)])
def test_3d_rows_on_both_sides_of_the_line(n_inst, iters):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng([n_inst, iters])
    b = W.Batch([W.make_3d3d(rng, 17, 0.01, 0.05, 512) for _ in range(n_inst)])
    gp = P.purse_default_params(n_iters=iters)
    res = PT.run_gpu(b, gp)
    g_radii, g_centre = rng.normal(size=(n_inst, 2)), rng.normal(size=(n_inst, 6))
    got, status = _grads(P, res, gp, 0, g_radii, g_centre)
    assert (status & 0xFF == P.PURSE_BWD_OK).all()
    ko = res["db"].kp_off_host
    grads, _ = _oracle(b, res, gp, n_inst - 1, g_radii, g_centre)
    assert _rel(got, ko[n_inst - 1], ko[n_inst], grads) <= RTOL
