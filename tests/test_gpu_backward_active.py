"""The backward's active set (the distinct samples of the trace and the first
feasible one) from traces made up here: its size against numpy's and its
status, from one member to beyond the capacity of 256, with ids spread over the
instance and with ids that crowd the last buckets of the hash table (and go
round its end)."""
import numpy as np
import pytest
import torch

from paper_2403_09990_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_backward_rev import _grads

pytestmark = pytest.mark.gpu


def _bucket(ids):
    return (ids.astype(np.uint64) * np.uint64(2654435761) & np.uint64(0xFFFFFFFF)) >> np.uint64(21)


@pytest.mark.parametrize("crowded", [False, True])
@pytest.mark.parametrize("members", [1, 2, 65, 254, 257, 600])
def test_active_set_of_a_given_trace(members, crowded):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng([members, crowded])
    b = W.Batch([W.make_3d3d(rng, 9, 0.01, 0.05, 30000)])
    gp = P.purse_default_params(n_iters=4)
    res = PT.run_gpu(b, gp)
    ok = np.nonzero(res["mask"].cpu().numpy() & P.PURSE_MASK_FEASIBLE)[0]
    pool = ok[1:][np.argsort(-_bucket(ok[1:]).astype(np.int64), kind="stable")] if crowded else rng.permutation(ok[1:])
    ids = np.concatenate([ok[:1], pool[:members - 1]])
    assert len(ids) == members
    T = gp.megb_iters
    tr = ids[rng.integers(0, members, size=2 * T)]
    tr[rng.choice(2 * T, size=members, replace=False)] = ids
    res["trace"] = torch.as_tensor(tr.reshape(1, T, 2), dtype=torch.int32, device="cuda").contiguous()
    got, status = _grads(P, res, gp, 0, np.ones((1, 2)), np.ones((1, 6)))
    assert status[0] >> 8 == members
    assert status[0] & 0xFF == (P.PURSE_BWD_OK if members < 256 else P.PURSE_BWD_OVERFLOW)
    assert all(np.isnan(g).all() if members > 256 else np.isfinite(g).all() for g in got[::2])
