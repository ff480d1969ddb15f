"""Remote 2D-3D anchors in a batch that holds many of them, at 300 instances and
at one more than the records a workgroup looks at in a round (512): an
instance's gradients are bitwise those of a call of its own."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import _grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_inst", [300, 513])
def test_remote_anchors_do_not_depend_on_the_batch(n_inst):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(n_inst)
    insts = [W.make_2d3d(rng, int(rng.integers(6, 25)), 2.0, (3.0, 6.0), 64) for _ in range(n_inst)]
    gp = P.purse_default_params(n_iters=40, kappa=0.9, megb_iters=128)
    res = PT.run_gpu(W.Batch(insts), gp)
    g_radii, g_centre = rng.normal(size=(n_inst, 2)), rng.normal(size=(n_inst, 6))
    got, _ = _grads(P, res, gp, 0, g_radii, g_centre)
    st, nf = res["inst_status"].cpu().numpy(), res["n_feasible"].cpu().numpy()
    js = [j for j in range(n_inst) if st[j] & P.PURSE_INST_ANCHOR_ITERATED
          and not st[j] & P.PURSE_INST_NO_ANCHOR and st[j] & 0xFF == P.PURSE_INST_OK and nf[j] > 0]
    assert len(js) > 8
    ko = res["db"].kp_off_host
    for j in js[:3] + js[-3:]:
        one = PT.run_gpu(W.Batch([insts[j]]), gp)
        alone, status = _grads(P, one, gp, 0, g_radii[j:j + 1], g_centre[j:j + 1])
        assert status[0] & 0xFF == P.PURSE_BWD_OK
        for a, c in zip(got, alone):
            assert np.array_equal(a[ko[j]:ko[j + 1]], c), j
