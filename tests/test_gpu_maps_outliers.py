"""MaskExtend on maps of every range: what a pixel gets depends on its own window
alone, however large the maps' values are elsewhere in the section, in the other
channels or in the other sections, and is as accurate as with the FP32 kernels.
Bar: rms error against 64 bits within 1.25 of the FP32 kernels', plus one output
rounding (2^-24), the sample's room in the other split tests."""
import numpy as np
import pytest

import oracle
from synth import maskextend_maps
from synth.nets import NET_ME, he_normal_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    assert torch.cuda.is_available()
    return m


def _ref(maps, p):
    return oracle.forward_maps(np.ascontiguousarray(np.transpose(maps, (0, 3, 1, 2)), dtype=np.float64), NET_ME, p)


def _nets(emcnn, p):
    """The net as a caller has it, and with an FP32 kernel chosen for every layer."""
    h, f = emcnn.cnn_create(p, NET_ME, "fp32"), emcnn.cnn_create(p, NET_ME, "fp32")
    for layer in range(5):
        names = [n for n in emcnn.cnn_variant_names(f, layer) if "<F32," in n]
        emcnn.cnn_set_variant(f, layer, names[0])
    return h, f


def _rms(got, ref):
    return float(np.sqrt(np.mean((got.cpu().numpy().astype(np.float64) - ref) ** 2)))


def _scaled(p, channels, exponent):
    """Weights for maps whose `channels` are 2^exponent times as large: the same function."""
    q = p.copy()
    q[:64 * 12 * 16].reshape(64, 12, 16)[:, channels] *= 2.0 ** -exponent
    return q


# EM sections as raw grey values beside masks and probabilities (255 = 2^8 nearly); all maps tiny;
# all large; one channel at the end of the range
@pytest.mark.parametrize("channels,exponent", [(slice(0, 3), 8), (slice(0, 12), -20), (slice(0, 12), 18), (slice(3, 4), 20)])
def test_channels_of_other_ranges(emcnn, channels, exponent):
    maps = maskextend_maps(34, 1, 140, 133)
    p = he_normal_params(NET_ME, 51)
    maps[..., channels] *= np.float32(2.0 ** exponent)
    q = _scaled(p, channels, exponent)
    ref = _ref(maps, q)
    h, f = _nets(emcnn, q)
    x = torch.from_numpy(maps).cuda()
    assert _rms(emcnn.cnn_infer_maps(h, x), ref) <= 1.25 * _rms(emcnn.cnn_infer_maps(f, x), ref) + 2.0 ** -24


@pytest.mark.parametrize("value", [2.0 ** 4, 255.0, 2.0 ** 12, -2.0 ** 20])
def test_an_outlier_changes_its_own_windows_only(emcnn, value):
    maps = maskextend_maps(35, 2, 150, 141)
    p = he_normal_params(NET_ME, 51)
    h, f = _nets(emcnn, p)
    x = torch.from_numpy(maps).cuda()
    base = emcnn.cnn_infer_maps(h, x).clone()
    odd = x.clone()
    odd[1, 3, 4, 5] = value  # in the windows of output rows 0..3 and columns 0..4
    got = emcnn.cnn_infer_maps(h, odd)
    assert torch.equal(got[0], base[0])
    assert torch.equal(got[1, 4:], base[1, 4:]) and torch.equal(got[1, :, 5:], base[1, :, 5:])
    ref = _ref(odd.cpu().numpy(), p)
    assert _rms(got, ref) <= 1.25 * _rms(emcnn.cnn_infer_maps(f, odd), ref) + 2.0 ** -24


def test_crops_beside_an_outlier(emcnn):
    maps = torch.from_numpy(maskextend_maps(36, 2, 170, 180)).cuda()
    maps[0, 160, 170, 2] = 2.0 ** 14
    h = emcnn.cnn_create(he_normal_params(NET_ME, 54), NET_ME, "fp32")
    full = emcnn.cnn_infer_maps(h, maps)
    for hh, ww in ((109, 109), (150, 180), (170, 150)):
        part = emcnn.cnn_infer_maps(h, maps[:, :hh, :ww].contiguous())
        assert torch.equal(part, full[:, :hh - 108, :ww - 108]), (hh, ww)
