"""A fallback call that cannot get its workspace fails before it enqueues anything."""
import pytest

from synth import em_volume
from synth.nets import NET_B, NET_S, calibrated_params, random_bias_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_a_call_without_memory_writes_nothing():
    import paper_1612_02120_amd as emcnn
    net = emcnn.cnn_create(calibrated_params("B"), NET_B, "fp32")
    s = emcnn.student_create(random_bias_params(NET_S, 317, 99, sigma=0.1), "bf16")
    # one slice whose inter-layer maps, 384 bytes a voxel, are larger than the device
    total = torch.cuda.get_device_properties(0).total_memory
    side = int((1.1 * total / 384) ** 0.5)
    vol = torch.zeros((1, side, side), dtype=torch.uint8, device="cuda")
    prob = torch.full((1, side - net.R, side - net.R), 7.0, device="cuda")
    with pytest.raises(emcnn.CnnError) as e:
        emcnn.student_infer_with_fallback(s, net, vol, tau=0.5, tile=1 << 20, n_samples=1, seed=5, out=prob)
    assert e.value.code == emcnn.CNN_ENOMEM
    torch.cuda.synchronize()
    assert bool((prob == 7.0).all())
    # the handles go on working
    small = torch.from_numpy(em_volume(112, 1, 60, 70)).cuda()
    out, _ = emcnn.student_infer_with_fallback(s, net, small, tau=-1.0, tile=16, n_samples=1, seed=5)
    assert torch.equal(out, emcnn.cnn_infer(net, small))
