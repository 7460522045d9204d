"""The walk over tiles that the fallback leaves to the student: more tiles than a
wave looks ahead over, closed ones in runs of every length, first and last ones
open or closed. Flagged tiles hold the teacher's map and the others the student's,
exactly (a voxel's arithmetic does not depend on the region that holds it)."""
import numpy as np
import pytest

from synth import em_volume
from synth.nets import NET_B, NET_S, calibrated_params, random_bias_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("teacher", ["fp32", "bf16"])
def test_flagged_tiles_among_many(teacher):
    import paper_1612_02120_amd as emcnn
    vol = torch.from_numpy(em_volume(111, 3, 300, 500)).cuda()
    net = emcnn.cnn_create(calibrated_params("B"), NET_B, teacher)
    s = emcnn.student_create(random_bias_params(NET_S, 316, 98, sigma=0.1), "bf16")
    T = emcnn.cnn_infer(net, vol)
    S = emcnn.student_infer(s, vol)[:, 3:-3, 3:-3]
    Z, Ho, Wo = T.shape
    ty, tx = emcnn.fallback_tiles(T.shape, 16)
    n = Z * ty * tx
    assert n > 8 * 64  # workgroups of one XCD walk an eighth of the tiles, 64 at a time where they are closed
    flags = torch.empty(n, dtype=torch.int32, device="cuda")
    seen = set()
    for tau in (-1.0, 0.0, 0.02, 0.1, 0.3, 0.6, 0.9, 2.0):
        out, st = emcnn.student_infer_with_fallback(s, net, vol, tau=tau, tile=16, n_samples=1, seed=5, flags=flags)
        torch.cuda.synchronize()
        m = flags.view(Z, ty, tx).bool().repeat_interleave(16, 1).repeat_interleave(16, 2)[:, :Ho, :Wo]
        assert torch.equal(out, torch.where(m, T, S)), tau
        seen.add(int(flags.sum()))
    assert 0 in seen and n in seen and len(seen) >= 4  # none, all, and several in between
