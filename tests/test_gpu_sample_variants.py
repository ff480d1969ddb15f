"""The sampler's launch variants give one another's samples bit for bit: small
batches in one launch with the tiles worked out in place, larger ones from the
device schedule, each kind in its own launch, and whole-wavefront or larger
workgroups; at the keypoint counts where its loops change (the unrolled loop's
end, held targets, groups of four records) and at the instance counts where the
schedule does."""
import numpy as np
import pytest
import torch

from paper_2403_09990_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(P, db, **kw):
    gp = P.purse_default_params(n_iters=12, **kw)
    ws = P.workspace(db, gp)
    ws.fill_(0xCD)
    poses = torch.full((db.total_samples, 12), float("nan"), dtype=torch.float32, device="cuda")
    mask = torch.full((db.total_samples,), 0xEE, dtype=torch.uint8, device="cuda")
    status = torch.full((db.n_inst,), -99, dtype=torch.int32, device="cuda")
    P.purse_sample(db, gp, poses, mask, status, ws)
    torch.cuda.synchronize()
    return poses.cpu(), mask.cpu(), status.cpu()


@pytest.mark.parametrize("n_inst", [1, 2, 63, 64, 65, 1025])
def test_launch_variants_agree_bitwise(n_inst):
    import paper_2403_09990_amd as P
    rng = np.random.default_rng(n_inst)
    n2, n3 = (6, 14, 15, 16, 17, 19, 20, 64), (3, 4, 5, 7, 8, 64)
    ins = []
    for j in range(n_inst):
        m = int(rng.integers(1, 200 if n_inst < 100 else 20))
        if (j + n_inst) % 2:
            ins.append(W.make_2d3d(rng, n2[(j // 2) % len(n2)], 2.0, (3.0, 25.0), m))
        else:
            ins.append(W.make_3d3d(rng, n3[(j // 2) % len(n3)], 0.01, (0.02, 0.1), m))
    db = P.DeviceBatch(W.Batch(ins))
    ref = _run(P, db, flags=P.PURSE_FLAG_SERIAL_GROUPS | P.PURSE_FLAG_INSTANCE_ORDER, tile=256)
    assert not torch.isnan(ref[0]).any() and not (ref[1] == 0xEE).any()
    for kw in (dict(), dict(tile=64), dict(tile=256), dict(flags=P.PURSE_FLAG_SERIAL_GROUPS),
               dict(flags=P.PURSE_FLAG_INSTANCE_ORDER), dict(flags=P.PURSE_FLAG_WORK_QUEUE),
               dict(waves_per_simd=2)):
        got = _run(P, db, **kw)
        assert all(torch.equal(a, b) for a, b in zip(got, ref)), kw
