"""GPU 3-D watershed (watershed_3d, through the C ABI) against the exact CPU
reference, label for label: the labelling is unique (a total order, no
flooding order), so the bar is bitwise equality. Cases: tiny volumes with many
exact ties, ragged sizes, every seed / no seed / one voxel, a synthetic 3-D
Voronoi map, and the membrane map of net B over an EM-like stack at full
headline size (32 x 1012 x 1012)."""
import numpy as np
import pytest
from scipy import ndimage  # noqa: E402

import oracle
from synth import em_volume
from synth.nets import NET_B, calibrated_params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emcnn():
    import paper_1612_02120_amd as m
    assert torch.cuda.is_available()
    return m


def _gpu(emcnn, p, t):
    lab = emcnn.watershed_3d(torch.from_numpy(np.ascontiguousarray(p)).cuda(), t)
    torch.cuda.synchronize()
    return lab.cpu().numpy()


@pytest.mark.parametrize("shape,levels,t,seed", [((3, 5, 6), 0, 0.2, 0), ((2, 7, 4), 4, 0.3, 1),
                                                 ((5, 37, 41), 6, 0.25, 2), ((1, 1, 1), 0, 0.5, 3),
                                                 ((4, 33, 65), 0, 2.0, 4), ((3, 40, 29), 3, -1.0, 5),
                                                 ((2, 64, 64), 1, 0.5, 6)])
def test_watershed_random_with_ties(emcnn, shape, levels, t, seed):
    print("watershed case", shape, levels, t, flush=True)
    rng = np.random.default_rng(seed)
    p = rng.uniform(0, 1, shape)
    if levels:
        p = np.floor(p * levels) / levels
    p = p.astype(np.float32)
    assert np.array_equal(_gpu(emcnn, p, t), oracle.watershed(p, t))


@pytest.mark.parametrize("shape,frac,seed", [((3, 9, 600), 0.85, 7), ((2, 5, 1030), 0.97, 8), ((2, 3, 700), 1.0, 9),
                                              ((4, 6, 257), 0.6, 10)])
def test_watershed_long_seed_runs(emcnn, shape, frac, seed):
    """Seed runs along x that cross the 256-column chunks of a row (the
    first-seed scan carries between chunks), rows that are all seeds, and
    exact ties among the seeds and the rest."""
    print("watershed runs case", shape, frac, flush=True)
    rng = np.random.default_rng(seed)
    p = np.floor(rng.uniform(0, 1, shape) * 5) / 5 + 0.2
    p = np.where(rng.uniform(0, 1, shape) < frac, 0.1, p).astype(np.float32)
    t = 0.15
    assert np.array_equal(_gpu(emcnn, p, t), oracle.watershed(p, t))


@pytest.mark.parametrize("sigma,q", [(1.0, 0.1), (2.5, 0.3)])
def test_watershed_smooth_maps(emcnn, sigma, q):
    rng = np.random.default_rng(11)
    p = ndimage.gaussian_filter(rng.uniform(0, 1, (9, 130, 117)), sigma).astype(np.float32)
    t = float(np.quantile(p, q))
    assert np.array_equal(_gpu(emcnn, p, t), oracle.watershed(p, t))


def test_watershed_on_net_b_map_full_size(emcnn):
    """The over-segmentation stage on the plain net's output over the headline
    volume (32 x 1024^2 in, 32 x 1012^2 map)."""
    h = emcnn.cnn_create(calibrated_params("B"), NET_B, "fp32")
    vol = torch.from_numpy(em_volume(2, 32, 1024, 1024)).cuda()
    pm = emcnn.cnn_infer(h, vol)
    t = float(torch.quantile(pm[0].flatten()[::97].float(), 0.25).item())
    lab = emcnn.watershed_3d(pm, t)
    torch.cuda.synchronize()
    P = pm.cpu().numpy()
    ref = oracle.watershed(P, t)
    got = lab.cpu().numpy()
    print("net B map %s, t %.4f: %d basins" % (P.shape, t, len(np.unique(ref))))
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("W", [1, 3, 4, 252, 255, 256, 257, 508, 512])
@pytest.mark.parametrize("offset", [0, 1])
def test_watershed_row_ends_and_alignment(emcnn, W, offset):
    """Rows that end inside a lane's four columns or a wave's 256, and maps that do
    not start at 16 bytes (read element by element), in one large component."""
    rng = np.random.default_rng(W)
    p = np.where(rng.uniform(0, 1, (3, 21, W)) < 0.7, 0.05, rng.uniform(0, 1, (3, 21, W))).astype(np.float32)
    flat = torch.empty(p.size + offset, dtype=torch.float32, device="cuda")
    view = flat[offset:].view(p.shape)
    view.copy_(torch.from_numpy(p))
    lab = emcnn.watershed_3d(view, 0.1)
    torch.cuda.synchronize()
    assert np.array_equal(lab.cpu().numpy(), oracle.watershed(p, 0.1))


@pytest.mark.parametrize("shape", [(2, 256, 256), (2, 256, 257), (3, 181, 290)])
def test_watershed_around_the_small_volume_form(emcnn, shape):
    """Volumes of 2^17 voxels and just above and beside it."""
    rng = np.random.default_rng(shape[2])
    p = ndimage.gaussian_filter(rng.uniform(0, 1, shape), 1.5).astype(np.float32)
    t = float(np.quantile(p, 0.4))
    assert np.array_equal(_gpu(emcnn, p, t), oracle.watershed(p, t))


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 8, 128), (3, 9, 129), (4, 17, 257), (1, 31, 127), (9, 2, 130),  # 2 x 8 x 128
                                   (5, 517, 413), (9, 257, 512), (4, 8, 33000)])  # 4 x 8 x 128
def test_watershed_across_tiles(emcnn, shape):
    """Volumes that end inside, at and past a tile, with seeds and ties through all faces."""
    print("watershed tiles case", shape, flush=True)
    rng = np.random.default_rng(shape[2])
    p = np.floor(rng.uniform(0, 1, shape) * 6) / 6
    p = np.where(rng.uniform(0, 1, shape) < 0.5, 0.05, p + 0.1).astype(np.float32)
    assert np.array_equal(_gpu(emcnn, p, 0.08), oracle.watershed(p, 0.08))


@pytest.mark.parametrize("H,W", [(300, 700), (800, 1500)])
def test_watershed_one_long_component(emcnn, H, W):
    """A seed path that winds through every tile: the deepest trees that tiles leave."""
    p = np.random.default_rng(H).uniform(0.2, 1, (1, H, W)).astype(np.float32)
    p[0, ::2] = 0.1
    p[0, 1::4, -1] = 0.1
    p[0, 3::4, 0] = 0.1
    assert np.array_equal(_gpu(emcnn, p, 0.15), oracle.watershed(p, 0.15))
