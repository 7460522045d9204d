"""The student's BF16 inference where its layout can go wrong: outputs narrower
than, at and past a strip of 62 columns, strips of few rows, odd last columns, and
an activation that is not finite beside the pixel pair that shares its window. Bar
as in test_gpu_student: 2e-3 to the reference with the same roundings."""
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


# outputs: 1 x 1; one column short of, at and past a strip and two; one row, one short of and past
# eight; more rows than the tallest strip (with enough strips for it: many slices)
@pytest.mark.parametrize("Z,Ho,Wo", [(1, 1, 1), (1, 1, 61), (2, 7, 62), (1, 9, 63), (3, 8, 64), (1, 17, 124), (1, 16, 125),
                                     (20, 260, 131)])
def test_inference_at_strip_edges(emcnn, Z, Ho, Wo):
    vol = em_volume(Ho + Wo, Z, Ho + 6, Wo + 6)
    p = random_bias_params(NET_S, 313, 74, sigma=0.1)
    buf = torch.full((Z * Ho * Wo + 64,), -7.0, device="cuda")  # what follows the output stays
    emcnn.student_infer(emcnn.student_create(p, "bf16"), torch.from_numpy(vol).cuda(),
                        out=buf[:Z * Ho * Wo].view(Z, Ho, Wo))
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert (got[Z * Ho * Wo:] == -7.0).all()
    got = got[:Z * Ho * Wo].reshape(Z, Ho, Wo)
    ref = oracle.forward(vol[-2:], NET_S, p, qmode="bf16")
    assert np.abs(got[-2:] - ref).max() <= 2e-3


def test_tall_strips_equal_short_ones(emcnn):
    # 4 x 1500^2 runs in strips of 32 rows or more, a crop of it in strips of 8: the same sums
    vol = torch.from_numpy(em_volume(75, 4, 1500, 1500)).cuda()
    s = emcnn.student_create(random_bias_params(NET_S, 314, 75, sigma=0.1), "bf16")
    whole = emcnn.student_infer(s, vol)
    part = emcnn.student_infer(s, vol[1:2, 700:900, 601:777].contiguous())
    assert torch.equal(whole[1:2, 700:894, 601:771], part)


def test_an_infinite_activation_reaches_only_its_own_outputs(emcnn):
    # h1 channel 0 overflows where the input is 255 and takes no part elsewhere (its W2 is 0)
    p = random_bias_params(NET_S, 315, 76, sigma=0.1)
    p[208:784].reshape(8, 8, 9)[:, 0] = 0.0
    ref_p = p.copy()
    w1 = p[:200].reshape(8, 25)
    w1[0] = 0.0
    w1[0, 24] = 3.0e38  # the last tap: input (y + 4, x + 4) for h1 (y, x)
    p[200] = 5.0e37
    vol = np.minimum(em_volume(76, 1, 60, 150), 200)
    hits = [(20, 8), (28, 17), (36, 66), (44, 67), (30, 128), (12, 129)]
    reached = np.zeros((54, 144), dtype=bool)
    for y, x in hits:
        vol[0, y, x] = 255
        reached[max(y - 6, 0):y - 3, max(x - 6, 0):x - 3] = True
    out = emcnn.student_infer(emcnn.student_create(p, "bf16"), torch.from_numpy(vol).cuda())
    torch.cuda.synchronize()
    got = out.cpu().numpy()[0]
    ref = oracle.forward(vol, NET_S, ref_p, qmode="bf16")[0]
    assert np.abs(got - ref)[~reached].max() <= 2e-3
