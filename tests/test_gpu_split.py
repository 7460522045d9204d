"""The FP32 convs on f16 hi/lo pairs (conv_split): parity with the FP64 oracle
at the edges of their tiles, no larger error than the FP32 MFMA kernels, weights
whose channels differ by many powers of two, and the rule that keeps a net whose
activations have no usable bound on the FP32 kernels."""
import numpy as np
import pytest
import torch

import oracle
from synth import em_volume, maskextend_maps
from synth.nets import (NET_A, NET_B, NET_FM, NET_FMSS, NET_ME, bias_slices, calibrated_params, he_normal_params,
                        random_bias_params)

pytestmark = pytest.mark.gpu

TOL = 1e-5  # the FP32 form's tolerance against the oracle, as in the parity tests


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    return m


def _run(emcnn, h, vol):
    out = emcnn.cnn_infer(h, torch.from_numpy(vol).cuda())
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _is_split(name):
    return name.startswith("conv_split<") or "<F32S," in name


# output sides: one pixel, one short of / exactly / one past a tile, several tiles
@pytest.mark.parametrize("net,R,shapes", [
    (NET_A, 8, [(1, 1, 1), (2, 15, 33), (1, 16, 32), (1, 17, 31), (3, 50, 70)]),
    (NET_B, 12, [(1, 1, 1), (1, 23, 33), (2, 24, 32), (1, 25, 31), (1, 16, 48), (1, 17, 49), (3, 60, 100)]),
    (NET_FM, 52, [(1, 1, 1), (1, 7, 9), (2, 64, 128), (1, 65, 127), (1, 70, 133)]),
], ids=["A", "B", "FM"])
def test_tile_edges_match_oracle_with_every_shape(emcnn, net, R, shapes):
    p = random_bias_params(net, 21, 22)
    h = emcnn.cnn_create(p, net, "fp32")
    n_body = sum(L["kind"] == "conv" and L["k"] > 1 for L in net) - 1
    for z, ho, wo in shapes:
        vol = em_volume(z + ho, z, ho + R, wo + R)
        ref = oracle.forward(vol, net, p)
        base = _run(emcnn, h, vol)
        assert np.abs(base - ref).max() <= TOL, (z, ho, wo)
        for layer in range(1, n_body + 1):
            names = emcnn.cnn_variant_names(h, layer)
            split = [n for n in names if _is_split(n)]
            assert names[0].startswith("head") or _is_split(names[0]), names[0]
            for name in split[1:]:  # the same K order: the same bits whatever the tile
                emcnn.cnn_set_variant(h, layer, name)
                assert np.array_equal(_run(emcnn, h, vol), base), (name, z, ho, wo)
            emcnn.cnn_set_variant(h, layer, names[0])


@pytest.mark.parametrize("net,side", [(NET_A, 260), (NET_B, 200), (NET_FM, 200), (NET_FMSS, 330)],
                         ids=["A", "B", "FM", "FMSS"])
def test_error_is_no_larger_than_the_fp32_kernels(emcnn, net, side):
    # rms error against 64 bits, every split layer against every FP32 layer; a
    # quarter and one output rounding of room for the sample
    p = he_normal_params(net, 31)
    vol = em_volume(9, 2, side, side + 7)
    ref = oracle.forward(vol, net, p)
    h = emcnn.cnn_create(p, net, "fp32")
    rms = lambda: float(np.sqrt(np.mean((_run(emcnn, h, vol) - ref) ** 2)))  # noqa: E731
    got = rms()
    changed = 0
    for layer in range(1, 8):
        names = emcnn.cnn_variant_names(h, layer)
        if names and _is_split(names[0]):
            emcnn.cnn_set_variant(h, layer, [n for n in names if not _is_split(n)][0])
            changed += 1
    assert changed
    assert got <= 1.25 * rms() + 2.0 ** -24


def _rescaled(net, p, exps):
    """The same function with hidden channel c of conv i scaled by 2^exps[i][c] and unscaled in conv i + 1."""
    q, off, prev, conv = p.copy(), 0, None, 0
    for L in net:
        if L["kind"] != "conv":
            continue
        n = L["cout"] * L["cin"] * L["k"] ** 2
        w = q[off:off + n].reshape(L["cout"], L["cin"], -1)
        if prev is not None:
            w *= 2.0 ** -prev[None, :, None]
        prev = exps[conv] if conv < len(exps) else None
        if prev is not None:
            w *= 2.0 ** prev[:, None, None]
            q[off + n:off + n + L["cout"]] *= 2.0 ** prev
        off, conv = off + n + L["cout"], conv + 1
    return q


def test_channels_of_very_different_scales(emcnn):
    # powers of two commute with ReLU and the max filter: the same function, with
    # activations from 2^-30 to 2^30 beside each other
    p = random_bias_params(NET_B, 41, 42)
    rng = np.random.default_rng(5)
    q = _rescaled(NET_B, p, [rng.integers(-30, 31, 48).astype(np.float64) for _ in range(2)])
    vol = em_volume(3, 1, 70, 90)
    h = emcnn.cnn_create(q, NET_B, "fp32")
    assert _is_split(emcnn.cnn_variant_names(h, 1)[0])
    assert np.abs(_run(emcnn, h, vol) - oracle.forward(vol, NET_B, p)).max() <= TOL


def test_unbounded_activations_keep_the_fp32_kernels(emcnn):
    vol = em_volume(4, 1, 40, 40)
    a, b = bias_slices(NET_B)[0]
    p = calibrated_params("B")
    p[a] = -1e37  # bias: a bound whose scale leaves the exponent range (the ReLU output itself is 0)
    h = emcnn.cnn_create(p, NET_B, "fp32")
    assert _is_split(emcnn.cnn_variant_names(h, 1)[0])  # the channel's bound is 0: scalable
    p[a] = 1e37
    h = emcnn.cnn_create(p, NET_B, "fp32")
    for layer in (1, 2):
        assert not any(_is_split(n) for n in emcnn.cnn_variant_names(h, layer))
    p[a] = np.inf
    h = emcnn.cnn_create(p, NET_B, "fp32")
    for layer in (1, 2):
        assert not any(_is_split(n) for n in emcnn.cnn_variant_names(h, layer))
    _run(emcnn, h, vol)


def _fp32_variants(emcnn, h, layers):
    for layer in range(layers):
        names = [n for n in emcnn.cnn_variant_names(h, layer) if not _is_split(n)]
        if names:
            emcnn.cnn_set_variant(h, layer, names[0])


def test_maskextend_split_error_and_scaled_maps(emcnn):
    maps = maskextend_maps(31, 2, 150, 141)
    p = he_normal_params(NET_ME, 51)
    ref = oracle.forward_maps(np.ascontiguousarray(np.transpose(maps, (0, 3, 1, 2)), dtype=np.float64), NET_ME, p)
    x = torch.from_numpy(maps).cuda()
    h = emcnn.cnn_create(p, NET_ME, "fp32")
    assert all(_is_split(emcnn.cnn_variant_names(h, layer)[0]) for layer in range(5))
    base = emcnn.cnn_infer_maps(h, x).cpu().numpy()
    assert np.abs(base - ref).max() <= TOL
    f = emcnn.cnn_create(p, NET_ME, "fp32")
    _fp32_variants(emcnn, f, 5)
    plain = emcnn.cnn_infer_maps(f, x).cpu().numpy()
    assert np.sqrt(np.mean((base - ref) ** 2)) <= 1.25 * np.sqrt(np.mean((plain - ref) ** 2)) + 2.0 ** -24
    # maps 2^9 times as large under weights 2^-9 times as large: the same function
    q = p.copy()
    q[:64 * 12 * 16] *= 2.0 ** -9
    hq = emcnn.cnn_create(q, NET_ME, "fp32")
    big = emcnn.cnn_infer_maps(hq, x * 512.0).cpu().numpy()
    assert np.abs(big - ref).max() <= TOL


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf"), 2.0 ** 30])
def test_maps_without_a_usable_range_take_the_fp32_kernels(emcnn, value):
    maps = torch.from_numpy(maskextend_maps(32, 2, 130, 125)).cuda()
    p = he_normal_params(NET_ME, 52)
    h, f = emcnn.cnn_create(p, NET_ME, "fp32"), emcnn.cnn_create(p, NET_ME, "fp32")
    _fp32_variants(emcnn, f, 5)
    before = emcnn.cnn_infer_maps(h, maps).clone()
    odd = maps.clone()
    odd[1, 3, 4, 5] = value
    a, b = emcnn.cnn_infer_maps(h, odd), emcnn.cnn_infer_maps(f, odd)
    torch.cuda.synchronize()
    assert torch.equal(torch.nan_to_num(a, nan=-1.0), torch.nan_to_num(b, nan=-1.0))
    # the next call starts from its own range
    assert torch.equal(emcnn.cnn_infer_maps(h, maps), before)


def test_maps_range_of_an_unaligned_tensor(emcnn):
    maps = torch.from_numpy(maskextend_maps(33, 1, 125, 121)).cuda()
    p = he_normal_params(NET_ME, 53)
    h = emcnn.cnn_create(p, NET_ME, "fp32")
    flat = torch.empty(maps.numel() + 4, dtype=torch.float32, device="cuda")
    for off in (0, 4):  # 16-byte steps: what the layers' own loads take
        view = flat[off:off + maps.numel()].view(maps.shape)
        view.copy_(maps)
        assert torch.equal(emcnn.cnn_infer_maps(h, view), emcnn.cnn_infer_maps(h, maps))
