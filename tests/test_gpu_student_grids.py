"""Launches past 2^32 threads along a side of the grid: tens of millions of patches or strips."""
import numpy as np
import pytest

import oracle
from synth import em_volume
from synth.nets import NET_S, random_bias_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [(1 << 20) + 8, (1 << 24) + 8])  # one block a patch of 7 x 7
def test_gradient_of_very_many_patches(B):
    import paper_1612_02120_amd as emcnn
    rng = np.random.default_rng(77)
    eight = em_volume(77, 1, 64, 64)[0][:56].reshape(8, 7, 64)[:, :, :7].copy()
    t8 = rng.uniform(0, 1, size=(8, 1, 1)).astype(np.float32)
    p = random_bias_params(NET_S, 311, 72, sigma=0.1)
    s = emcnn.student_create(p, "fp32")
    patches = torch.from_numpy(eight).cuda().repeat(B // 8, 1, 1)
    target = torch.from_numpy(t8).cuda().repeat(B // 8, 1, 1)
    g, loss = emcnn.student_grad(s, patches, target)
    g = g.cpu().numpy().astype(np.float64)
    lref, gref = oracle.student_loss_grad(eight, t8.astype(np.float64), NET_S, p)
    # the mean over B patches is that over eight; 9 B / 2048 partial sums are added one after another in FP32
    room = 1e-4 + 9 * B / 2048 * 2.0 ** -24
    assert abs(loss.item() - lref) <= 1e-6 * abs(lref)
    assert np.abs(g - gref).max() <= room * np.abs(gref).max()


def test_student_over_very_many_strips():
    import paper_1612_02120_amd as emcnn
    Z, W = 65535, 62 * 1024 + 7  # 1025 strips of 62 columns a slice of one output row
    s = emcnn.student_create(random_bias_params(NET_S, 318, 97, sigma=0.1), "bf16")
    row = torch.randint(0, 256, (7, W), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    one = emcnn.student_infer(s, row[None].contiguous())
    out = emcnn.student_infer(s, row.expand(Z, 7, W).contiguous())
    assert torch.equal(out, one.expand(Z, 1, W - 6))
