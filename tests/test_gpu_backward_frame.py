"""The tangents of the centre and the anchor against the oracle: a centre fit
that converged (differentiated at its fixed point), one stopped by its cap
(re-run from its start), the closed 3D-3D form, and 3D-3D anchors that an
iteration had to find."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import RTOL, _grads, _oracle, _rel

pytestmark = pytest.mark.gpu


def _check(b, gp, js=None):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(5)
    res = PT.run_gpu(b, gp)
    g_radii, g_centre = rng.normal(size=(b.n_inst, 2)), rng.normal(size=(b.n_inst, 6))
    got, status = _grads(P, res, gp, 0, g_radii, g_centre)
    ko = res["db"].kp_off_host
    for j in range(b.n_inst) if js is None else js(res):
        assert status[j] & 0xFF == P.PURSE_BWD_OK
        grads, _ = _oracle(b, res, gp, j, g_radii, g_centre)
        assert _rel(got, ko[j], ko[j + 1], grads) <= RTOL, j


@pytest.mark.parametrize("kind,n_kp,centre_gn", [("2d", 6, 50), ("2d", 17, 50), ("2d", 17, 2), ("3d", 3, 50),
                                                 ("3d", 64, 50)])
def test_frame_tangents_match_oracle(kind, n_kp, centre_gn):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng([n_kp, centre_gn])
    inst = W.make_2d3d(rng, n_kp, 2.0, (5.0, 20.0), 512) if kind == "2d" else W.make_3d3d(rng, n_kp, 0.01, 0.05, 512)
    _check(W.Batch([inst]), P.purse_default_params(n_iters=20, centre_gn=centre_gn))


def test_iterated_anchor_tangents_match_oracle():
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(6)
    b = W.Batch([W.make_3d3d(rng, int(rng.integers(6, 49)), 0.01, (0.02, 0.1), 256) for _ in range(512)])

    def remote(res):
        st = res["inst_status"].cpu().numpy()
        nf = res["n_feasible"].cpu().numpy()
        js = [j for j in range(b.n_inst) if st[j] & P.PURSE_INST_ANCHOR_ITERATED
              and not st[j] & P.PURSE_INST_NO_ANCHOR and st[j] & 0xFF == P.PURSE_INST_OK and nf[j] > 0]
        assert js, "no instance with an iterated anchor"
        return js[:2]
    _check(b, P.purse_default_params(n_iters=20), remote)
