"""Tangents of remote 2D-3D anchors (the centre not inside the shrunk set, so
the anchor is the end of a trajectory from it) against the oracle: such
instances are rare, so they are looked for among 8,192 small ones."""
import numpy as np
import pytest

from paper_2403_09990_amd import workloads as W
from tests.test_gpu_backward_frame import _check

pytestmark = pytest.mark.gpu


def test_remote_2d_anchor_tangents_match_oracle():
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(3)
    b = W.Batch([W.make_2d3d(rng, int(rng.integers(6, 49)), 2.0, (5.0, 20.0), 64) for _ in range(8192)])

    def remote(res):
        st = res["inst_status"].cpu().numpy()
        nf = res["n_feasible"].cpu().numpy()
        js = [j for j in range(b.n_inst) if st[j] & P.PURSE_INST_ANCHOR_ITERATED
              and not st[j] & P.PURSE_INST_NO_ANCHOR and st[j] & 0xFF == P.PURSE_INST_OK and nf[j] > 0]
        assert js, "no instance with a remote anchor"
        return js[:2]
    _check(b, P.purse_default_params(n_iters=20), remote)
