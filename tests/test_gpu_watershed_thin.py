"""Volumes with very many tiles: a few voxels a slice, tens of millions of slices."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Z", [4 * (1 << 20) + 3, 4 * (1 << 23) + 7])  # just past 2^20 tiles (one row of the grid) and 2^23
def test_more_tiles_than_one_row_of_a_grid(Z):
    import paper_1612_02120_amd as emcnn
    # slabs of four slices of seeds between single slices above the threshold: one label a slab, and a
    # slice between goes to the slab before it (equal values: the least index)
    z = torch.arange(Z, device="cuda")
    p = torch.where(z % 5 == 4, 0.5, 0.1).to(torch.float32)[:, None, None].expand(Z, 2, 2).contiguous()
    lab = emcnn.watershed_3d(p, 0.2)
    want = ((z // 5) * 20 + 1).to(torch.int32)[:, None, None].expand(Z, 2, 2)
    assert torch.equal(lab, want)
