"""Weight gradients beside an activation that is not finite, where the columns that a
stage carries over from the one before, or that a chunk starts with, hold it: an
infinite h1 past a row's outputs must reach no tap that does not read it."""
import numpy as np
import pytest

from synth.nets import NET_S, random_bias_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# h1 (y, x) of patch b is infinite, x just past the outputs of its row. (1, 128): the first column of
# a stage of 256 in the sixth chunk of 2048 positions, for filter rows 0..2 in turn. (215, 13): the
# second column that the sixth chunk starts with.
@pytest.mark.parametrize("B,P,b,y,x", [(1, 128, 0, 85, 122), (1, 128, 0, 86, 122), (1, 128, 0, 87, 122),
                                       (215, 13, 208, 6, 7)])
def test_an_infinite_activation_at_a_stage_start(B, P, b, y, x):
    import paper_1612_02120_amd as emcnn
    p = random_bias_params(NET_S, 312, 73, sigma=0.1)
    w1 = p[:200].reshape(8, 25)
    w1[0] = 0.0
    w1[0, 24] = 3.0e38  # the last tap: h1 (y, x) of channel 0 reads input (y + 4, x + 4)
    p[200] = 1.0e38
    p[208:784].reshape(8, 8, 9)[:, 0] = 0.0  # 0 times finite: the channel takes no part elsewhere
    patches = np.full((B, P, P), 20, dtype=np.uint8)
    patches[b, y + 4, x + 4] = 255
    t = np.full((B, P - 6, P - 6), 0.5, dtype=np.float32)
    s = emcnn.student_create(p, "fp32")
    g, _ = emcnn.student_grad(s, torch.from_numpy(patches).cuda(), torch.from_numpy(t).cuda())
    torch.cuda.synchronize()
    g2 = g.cpu().numpy()[208:784].reshape(8, 8, 3, 3)
    # tap (i, j) of W2[., 0] reads h1 (y, x) at output (y - i, x - j)
    reads = np.zeros((3, 3), dtype=bool)
    for i in range(3):
        for j in range(3):
            reads[i, j] = 0 <= y - i < P - 6 and 0 <= x - j < P - 6
    assert reads.any() and not reads.all()
    assert not np.isfinite(g2[:, 0][:, reads]).any()
    assert np.isfinite(g2[:, 0][:, ~reads]).all() and np.isfinite(g2[:, 1:]).all()
