"""Choices that an autotune cache holds from before the present kernels: a kernel that
rounds otherwise than the default is tuned anew, one that does not is taken."""
import pytest

from synth import em_volume
from synth.nets import NET_B, NET_FM, calibrated_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _is_split(name):
    return name.startswith("conv_split<") or "<F32S," in name


@pytest.mark.parametrize("name", ["B", "FM"])
def test_an_older_cache_does_not_choose_the_fp32_kernels(name, tmp_path):
    import paper_1612_02120_amd as emcnn
    net, layers = NET_B if name == "B" else NET_FM, (1, 2)
    p = calibrated_params(name)
    cache = tmp_path / "tuned.txt"
    vol = torch.from_numpy(em_volume(14, 1, 160, 160)).cuda()
    h = emcnn.cnn_create(p, net, "fp32")
    base = emcnn.cnn_infer(h, vol)
    emcnn.cnn_autotune(h, 160, 160, str(cache))
    lines = cache.read_text().splitlines()
    tuned = [line.rsplit("|", 1)[1] for line in lines]
    # the same file as a library without the split kernels wrote it, all lines but the split layers' as they are
    old = []
    for line in lines:
        key, chosen = line.rsplit("|", 1)
        for layer in layers:
            names = emcnn.cnn_variant_names(h, layer)
            if chosen in names and _is_split(chosen):
                chosen = [n for n in names if not _is_split(n)][0]
                break
        old.append(key + "|" + chosen)
    assert old != lines
    cache.write_text("\n".join(old) + "\n")
    g = emcnn.cnn_create(p, net, "fp32")
    emcnn.cnn_autotune(g, 160, 160, str(cache))
    assert torch.equal(emcnn.cnn_infer(g, vol), base)
    again = [line.rsplit("|", 1)[1] for line in cache.read_text().splitlines()]
    assert [_is_split(n) for n in again] == [_is_split(n) for n in tuned]
    # what the file holds now is taken as it is
    kept = cache.read_text()
    f = emcnn.cnn_create(p, net, "fp32")
    emcnn.cnn_autotune(f, 160, 160, str(cache))
    assert cache.read_text() == kept
    for n in dict(line.rsplit("|", 1) for line in kept.splitlines()).values():
        assert n in emcnn.cnn_describe(f)
