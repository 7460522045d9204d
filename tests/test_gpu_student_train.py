"""The student's training kernels where their layout can go wrong: patches at the
edges of the 16 x 32 forward tiles, rows shorter than a group of columns, chunks
of 2048 positions that end inside a row or a patch, and an activation that is
not finite beside a row's end. Bars as in test_gpu_student: FP32 gradients within
1e-4 of the largest, the loss within 1e-6."""
import numpy as np
import pytest

import oracle
from synth import em_volume
from synth.nets import NET_S, random_bias_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    assert torch.cuda.is_available()
    return m


# (P - 4) x (P - 4) h1 positions: 3 x 3; one tile row / column short of, at and past a tile; many
# short rows per chunk; one patch over several chunks; chunks ending inside a patch
@pytest.mark.parametrize("B,P", [(1, 7), (1, 19), (1, 20), (2, 21), (1, 36), (3, 37), (300, 8), (61, 13), (1, 100), (5, 61)])
def test_gradient_and_loss_at_tile_and_chunk_edges(emcnn, B, P):
    rng = np.random.default_rng(B * 1000 + P)
    patches = em_volume(B + P, 1, 260, 260)[0]
    at = rng.integers(0, 260 - P + 1, size=(B, 2))
    patches = np.stack([patches[y:y + P, x:x + P] for y, x in at])
    t = rng.uniform(0, 1, size=(B, P - 6, P - 6)).astype(np.float32)
    p = random_bias_params(NET_S, 311, 72, sigma=0.1)
    s = emcnn.student_create(p, "fp32")
    g, loss = emcnn.student_grad(s, torch.from_numpy(patches).cuda(), torch.from_numpy(t).cuda())
    torch.cuda.synchronize()
    lref, gref = oracle.student_loss_grad(patches, t.astype(np.float64), NET_S, p)
    g = g.cpu().numpy().astype(np.float64)
    assert abs(loss.item() - lref) <= 1e-6 * abs(lref)
    assert np.abs(g - gref).max() <= 1e-4 * np.abs(gref).max()


def test_an_infinite_activation_reaches_only_its_own_taps(emcnn):
    # h1 channel 0 overflows at the last column of the first row only. Tap (0, 2)
    # of W2[., 0] reads it (0 or a finite gradient times inf); taps j = 0, 1 never
    # do, nor do the other input channels or filter rows 1 and 2.
    P = 30
    p = random_bias_params(NET_S, 312, 73, sigma=0.1)
    w1 = p[:200].reshape(8, 25)
    w1[0] = 0.0
    w1[0, 24] = 3.0e38  # the last tap: input (4, P - 1) for h1 (0, P - 5)
    p[200] = 1.0e38
    patches = np.full((1, P, P), 20, dtype=np.uint8)
    patches[0, 4, P - 1] = 255
    t = np.full((1, P - 6, P - 6), 0.5, dtype=np.float32)
    p[208:784].reshape(8, 8, 9)[:, 0] = 0.0  # 0 times finite: the channel takes no part elsewhere
    s = emcnn.student_create(p, "fp32")
    g, _ = emcnn.student_grad(s, torch.from_numpy(patches).cuda(), torch.from_numpy(t).cuda())
    torch.cuda.synchronize()
    g2 = g.cpu().numpy()[208:784].reshape(8, 8, 3, 3)
    assert not np.isfinite(g2[:, 0, 0, 2]).any()
    rest = g2.copy()
    rest[:, 0, 0, 2] = 0.0
    assert np.isfinite(rest).all()
