"""The radius samples of the backward, searched by one workgroup per instance
in calls below 32,768 samples and spread over many above: an instance's
gradients are bitwise those of a call of its own that takes the other route,
and the large instance's match the oracle (at the line, one sample past it, and
with more rounds of 1,024 samples than the 256 workgroups)."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import RTOL, _grads, _oracle, _rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("big", [32768, 32769, 262145])
def test_radius_search_on_both_sides_of_the_line(big):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(big)
    insts = [W.make_2d3d(rng, 9, 2.0, (5.0, 20.0), 777), W.make_3d3d(rng, 11, 0.01, 0.05, 32767),
             W.make_2d3d(rng, 12, 2.0, (5.0, 20.0), big)]
    gp = P.purse_default_params(n_iters=10)
    g_radii, g_centre = rng.normal(size=(3, 2)), rng.normal(size=(3, 6))
    b = W.Batch(insts)
    res = PT.run_gpu(b, gp)
    got, status = _grads(P, res, gp, 0, g_radii, g_centre)
    assert (status & 0xFF == P.PURSE_BWD_OK).all()
    ko = res["db"].kp_off_host
    for j in (0, 1):
        one = PT.run_gpu(W.Batch([insts[j]]), gp)
        alone, _ = _grads(P, one, gp, 0, g_radii[j:j + 1], g_centre[j:j + 1])
        for a, c in zip(got, alone):
            assert np.array_equal(a[ko[j]:ko[j + 1]], c)
    grads, _ = _oracle(b, res, gp, 2, g_radii, g_centre)
    assert _rel(got, ko[2], ko[3], grads) <= RTOL
