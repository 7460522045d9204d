"""The tile shapes that a launch picks by its size change no bit: the map of a
small volume is the crop of a larger one's, whose layers run with other shapes,
for every net and precision; and a batch of small blocks, whose launches see all
blocks at once, equals the blocks one by one."""
import numpy as np
import pytest
import torch

from synth import em_volume
from synth.nets import NET_A, NET_B, NET_FM, NET_FMSS, NET_ME, fp8_act_scales, he_normal_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    return m


def _net(emcnn, net, prec):
    return emcnn.cnn_create(he_normal_params(net, 61), net, prec,
                            act_scales=fp8_act_scales("B") if prec == "fp8" else None)


# output sides from one pixel to several tiles of every shape; the large volume has 700^2 x 4
@pytest.mark.parametrize("net,prec", [(NET_A, "fp32"), (NET_B, "fp32"), (NET_B, "bf16"), (NET_B, "fp8"), (NET_FM, "fp32"),
                                      (NET_FM, "bf16"), (NET_FMSS, "fp32"), (NET_FMSS, "bf16")],
                         ids=["A", "B32", "B16", "B8", "FM32", "FM16", "FMSS32", "FMSS16"])
def test_small_volumes_are_crops_of_a_large_one(emcnn, net, prec):
    h = _net(emcnn, net, prec)
    vol = torch.from_numpy(em_volume(12, 4, 760, 700)).cuda()
    full = emcnn.cnn_infer(h, vol)
    for z, hh, ww in [(1, h.R + 1, h.R + 1), (1, h.R + 9, h.R + 17), (1, 130, 251), (2, 200, 160), (1, 333, 500),
                      (3, 410, 700)]:
        if hh <= h.R or ww <= h.R:
            continue
        out = emcnn.cnn_infer(h, vol[:z, :hh, :ww].contiguous())
        assert torch.equal(out, full[:z, :out.shape[1], :out.shape[2]]), (z, hh, ww)


def test_small_maps_are_crops_of_larger_ones(emcnn):
    h = _net(emcnn, NET_ME, "fp32")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    maps = torch.rand((3, 400, 420, 12), device="cuda", generator=g)
    full = emcnn.cnn_infer_maps(h, maps)
    for z, hh, ww in [(1, 109, 109), (1, 150, 133), (2, 260, 300)]:
        part = maps[:z, :hh, :ww].contiguous()
        out = emcnn.cnn_infer_maps(h, part)
        assert torch.equal(out, full[:z, :out.shape[1], :out.shape[2]]), (z, hh, ww)


@pytest.mark.parametrize("net,prec", [(NET_B, "fp32"), (NET_B, "bf16"), (NET_B, "fp8"), (NET_FM, "fp32"), (NET_FM, "bf16")],
                         ids=["B32", "B16", "B8", "FM32", "FM16"])
def test_batches_of_every_size_equal_their_blocks(emcnn, net, prec):
    h = _net(emcnn, net, prec)
    rng = np.random.default_rng(4)
    for n in (1, 3, 40):
        tiles = []
        for i in range(n):
            z, a, b = int(rng.integers(1, 3)), int(rng.integers(1, 90)), int(rng.integers(1, 120))
            v = torch.from_numpy(em_volume(100 + i, z, a + h.R, b + h.R)).cuda()
            tiles.append((v, h.R // 2, torch.empty((z, a, b), device="cuda")))
        emcnn.cnn_infer_batch(h, tiles)
        for v, _, out in tiles:
            assert torch.equal(out, emcnn.cnn_infer(h, v)), (n, tuple(out.shape))


def test_a_chosen_variant_stays(emcnn):
    h = _net(emcnn, NET_B, "fp32")
    vol = torch.from_numpy(em_volume(13, 1, 100, 100)).cuda()
    base = emcnn.cnn_infer(h, vol)
    old = [n for n in emcnn.cnn_variant_names(h, 1) if n.startswith("conv_mfma<")][0]
    emcnn.cnn_set_variant(h, 1, old)
    assert old in emcnn.cnn_describe(h)
    other = emcnn.cnn_infer(h, vol)
    assert not torch.equal(other, base)  # the FP32 MFMA's own rounding: it really ran
    emcnn.cnn_set_variant(h, 1, emcnn.cnn_variant_names(h, 1)[0])
    assert torch.equal(emcnn.cnn_infer(h, vol), base)
