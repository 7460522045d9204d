"""The rule that keeps a layer on the FP32 kernels where its weights and bounds
leave an f16 pair too few bits for its ordinary channels (conv_split): a hidden
channel that could reach far past the others and hardly ever does. Bar: rms error
against 64 bits within 1.25 of the FP32 kernels', plus one output rounding (2^-24)."""
import numpy as np
import pytest

import oracle
from synth import em_volume
from synth.nets import NET_B, NET_FM, NET_FMSS, calibrated_params, he_normal_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    assert torch.cuda.is_available()
    return m


def _is_split(name):
    return name.startswith("conv_split<") or "<F32S," in name


def _rms(emcnn, h, vol, ref):
    got = emcnn.cnn_infer(h, torch.from_numpy(vol).cuda()).cpu().numpy().astype(np.float64)
    return float(np.sqrt(np.mean((got - ref) ** 2)))


def _no_larger(emcnn, p, net, vol):
    ref = oracle.forward(vol, net, p)
    h = emcnn.cnn_create(p, net, "fp32")
    got = _rms(emcnn, h, vol, ref)
    for layer in range(1, 6):
        fp32 = [n for n in emcnn.cnn_variant_names(h, layer) if not _is_split(n)]
        if fp32:
            emcnn.cnn_set_variant(h, layer, fp32[0])
    assert got <= 1.25 * _rms(emcnn, h, vol, ref) + 2.0 ** -24


def _rare_channel(p, reach):
    """Channel 0 of net B's first conv: zero unless the window is a sharp checkerboard, then up to `reach`."""
    s = np.where(np.arange(25) % 2 == 0, 1.0, -1.0)
    a = reach / (13 * 0.01)
    p[:25] = a * s
    p[48 * 25] = -a * 13 * 0.99
    return p


@pytest.mark.parametrize("reach", [1e2, 1e4, 1e6, 1e8, 1e9, 1e12])
def test_a_large_channel_that_never_fires(emcnn, reach):
    _no_larger(emcnn, _rare_channel(calibrated_params("B"), reach), NET_B, em_volume(6, 1, 90, 100))


@pytest.mark.parametrize("n", [2, 13, 30, 47])
@pytest.mark.parametrize("reach", [1e6, 1e10])
def test_many_large_channels_that_never_fire(emcnn, n, reach):
    p = calibrated_params("B")
    s = np.where(np.arange(25) % 2 == 0, 1.0, -1.0)
    a = reach / (13 * 0.01)
    p[:25 * n].reshape(n, 25)[:] = a * s
    p[48 * 25:48 * 25 + n] = -a * 13 * 0.99
    _no_larger(emcnn, p, NET_B, em_volume(6, 1, 90, 100))


@pytest.mark.parametrize("n", [1, 9, 20, 32])
@pytest.mark.parametrize("reach", [1e6, 1e10])
def test_large_members_of_max_out_pairs_that_never_show(emcnn, n, reach):
    # FastMemb's first conv: the second member of n pairs is far below the first except on a sharp checkerboard
    p = calibrated_params("FM")
    s = np.where(np.add.outer(np.arange(4), np.arange(4)).reshape(16) % 2 == 0, 1.0, -1.0)
    a = reach / (8 * 0.01)
    p[:64 * 16].reshape(64, 16)[1:2 * n:2] = a * s
    p[64 * 16:64 * 17][1:2 * n:2] = -a * 8 * 0.99
    _no_larger(emcnn, p, NET_FM, em_volume(9, 1, 110, 100))


@pytest.mark.parametrize("n", [1, 13, 30, 47])
@pytest.mark.parametrize("scale", [1e4, 1e8])
def test_large_hidden_channels_that_never_fire(emcnn, n, scale):
    # the second conv's channels 0 .. n - 1: ordinary filters `scale` times as large, biases half as far
    # again below zero as the image raises them
    p = calibrated_params("B")
    vol = em_volume(10, 1, 90, 100)
    w1 = torch.from_numpy(p[:1200].reshape(48, 1, 5, 5))
    w2 = p[1248:1248 + 48 * 1200].reshape(48, 48, 5, 5)
    h = torch.relu(torch.nn.functional.conv2d(torch.from_numpy(vol[:, None] / 255.0), w1))
    z = torch.nn.functional.conv2d(torch.nn.functional.max_pool2d(h, 2, 1), torch.from_numpy(w2.copy()))
    w2[:n] *= scale
    p[1248 + 48 * 1200:1248 + 48 * 1200 + n] = -1.5 * scale * np.maximum(z.amax((0, 2, 3)).numpy()[:n], 1.0)
    _no_larger(emcnn, p, NET_B, vol)


@pytest.mark.parametrize("net", [NET_B, NET_FM], ids=["B", "FM"])
@pytest.mark.parametrize("rows", [1, 20, 47])
def test_filters_far_below_their_rows(emcnn, net, rows):
    # input channels of the second conv whose filters are 2^-20 of the others' (bounds alike)
    p = he_normal_params(net, 71)
    first, cin = (48 * 26, 48) if net is NET_B else (64 * 17, 32)
    k2, cout = (25, 48) if net is NET_B else (16, 64)
    w = p[first:first + cout * cin * k2].reshape(cout, cin, k2)
    w[:, :min(rows, cin - 1)] *= 2.0 ** -20
    _no_larger(emcnn, p, net, em_volume(7, 1, 100, 90))


@pytest.mark.parametrize("net", [NET_B, NET_FM, NET_FMSS], ids=["B", "FM", "FMSS"])
def test_images_of_the_darkest_grey_levels(emcnn, net):
    # levels 0 and 1: activations a hundredth of what their scales allow for
    _no_larger(emcnn, he_normal_params(net, 72), net, em_volume(8, 1, 130, 140) // 150)


def test_ordinary_nets_keep_the_split_kernels(emcnn):
    for net, p in ((NET_B, calibrated_params("B")), (NET_FM, calibrated_params("FM"))):
        h = emcnn.cnn_create(p, net, "fp32")
        assert all(_is_split(emcnn.cnn_variant_names(h, layer)[0]) for layer in (1, 2))


# filters of widely different norms; output channels of widely different norms; four of five weights
# zero; a fifth of the filters decayed to nothing; biases as large as the sums
@pytest.mark.parametrize("kind", ["filters", "channels", "sparse", "decayed", "biased"])
@pytest.mark.parametrize("net", [NET_B, NET_FM, NET_FMSS], ids=["B", "FM", "FMSS"])
def test_weights_of_other_distributions(emcnn, kind, net):
    for seed in (1, 2):
        rng = np.random.default_rng(seed)
        p, off = he_normal_params(net, 80 + seed), 0
        for L in net:
            if L["kind"] != "conv":
                continue
            n = L["cout"] * L["cin"] * L["k"] ** 2
            w = p[off:off + n].reshape(L["cout"], L["cin"], -1)
            if kind == "filters":
                w *= np.exp(rng.normal(0, 1.0, (L["cout"], L["cin"], 1)))
            elif kind == "channels":
                w *= np.exp(rng.normal(0, 1.5, (L["cout"], 1, 1)))
            elif kind == "sparse":
                w *= rng.uniform(size=w.shape) < 0.2
            elif kind == "decayed":
                w *= np.where(rng.uniform(size=(L["cout"], L["cin"], 1)) < 0.2, 1e-6, 1.0)
            elif L["cin"] > 1 and L["k"] > 1:
                p[off + n:off + n + L["cout"]] = rng.normal(0, 1.0, L["cout"])
            off += n + L["cout"]
        _no_larger(emcnn, p, net, em_volume(20 + seed, 1, 130, 140))
