"""The bounds behind the FP32 convs on f16 pairs (conv_split): nets whose bounds
nearly cancel, where only rounding is left of a channel, stay finite and right."""
import numpy as np
import pytest

import oracle
from synth import em_volume
from synth.nets import NET_B, calibrated_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-5  # the FP32 form's tolerance against the oracle, as in the parity tests


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    assert torch.cuda.is_available()
    return m


# 25 equal weights and a bias that cancels their sum exactly, or all but a residual
@pytest.mark.parametrize("weight", [0.04, 0.07, 0.013])
@pytest.mark.parametrize("residual", [0.0, 1e-9, -1e-9, 1e-7])
def test_a_channel_whose_bound_cancels(emcnn, weight, residual):
    p = calibrated_params("B")
    p[:25] = weight
    p[48 * 25] = -25 * weight + residual
    vol = em_volume(5, 2, 40, 44)
    vol[0] = 255
    vol[1, :20] = 255
    h = emcnn.cnn_create(p, NET_B, "fp32")
    got = emcnn.cnn_infer(h, torch.from_numpy(vol).cuda()).cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    assert np.abs(got - oracle.forward(vol, NET_B, p)).max() <= TOL


# the same in the second conv: its whole bound cancels, its FP32 sum does not
def test_a_hidden_channel_whose_bound_cancels(emcnn):
    p = calibrated_params("B")
    p[:48 * 25] = 0.04  # first conv: every channel reaches exactly its bound on white
    p[48 * 25:48 * 26] = 0.0
    w2 = p[48 * 26:48 * 26 + 48 * 48 * 25].reshape(48, 48 * 25)
    w2[0] = 0.01
    p[48 * 26 + 48 * 48 * 25] = -12.0
    vol = np.full((1, 40, 40), 255, dtype=np.uint8)
    h = emcnn.cnn_create(p, NET_B, "fp32")
    got = emcnn.cnn_infer(h, torch.from_numpy(vol).cuda()).cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    assert np.abs(got - oracle.forward(vol, NET_B, p)).max() <= TOL
