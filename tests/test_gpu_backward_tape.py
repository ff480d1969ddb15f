"""The reverse sweeps against the oracle on either side of what their tape
keeps: the factors of the 2D-3D passes while the rows fit a compute unit's LDS
and the call is small (134 iterations of two passes, not 135; not in a batch of
five), and the 3D-3D targets' matrices while they fit 64 KB (146 iterations,
not 147)."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import RTOL, _grads, _oracle, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n_inst,iters", [("2d", 1, 134), ("2d", 1, 135), ("2d", 5, 20), ("3d", 1, 146),
                                               ("3d", 1, 147)])
def test_reverse_sweep_on_both_sides_of_the_tape(kind, n_inst, iters):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng([n_inst, iters])
    make = (lambda: W.make_2d3d(rng, 17, 2.0, (5.0, 20.0), 1024)) if kind == "2d" else (
        lambda: W.make_3d3d(rng, 17, 0.01, 0.05, 1024))
    b = W.Batch([make() for _ in range(n_inst)])
    gp = P.purse_default_params(n_iters=iters)
    res = PT.run_gpu(b, gp)
    g_radii, g_centre = rng.normal(size=(n_inst, 2)), rng.normal(size=(n_inst, 6))
    got, status = _grads(P, res, gp, 0, g_radii, g_centre)
    assert (status & 0xFF == P.PURSE_BWD_OK).all()
    ko = res["db"].kp_off_host
    grads, _ = _oracle(b, res, gp, n_inst - 1, g_radii, g_centre)
    assert _rel(got, ko[n_inst - 1], ko[n_inst], grads) <= RTOL
