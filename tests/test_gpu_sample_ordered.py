"""Trilinear samples of a VDB at ordered positions and past the volume, where a
wave's lanes share leaves: equal bit for bit to the samples of the reconstructed
volume as a plain array, and the same every time.  The volume reaches over the
borders of lower nodes (128 voxels) and has constant regions at both levels."""
import numpy as np
import pytest
import torch

from paper_2504_04564_amd import _build, vdbc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scene():
    _build.ensure_built()
    rng = np.random.default_rng(6)
    v = rng.random((150, 139, 272), dtype=np.float32)
    empty = rng.random((19, 18, 34)) < 0.5   # leaf regions of the background
    v[np.kron(empty, np.ones((8, 8, 8), bool))[:150, :139, :272]] = 0.0
    v[:128, :128, 128:256] = 0.5        # an upper tile
    v[129:145, 8:24, 100:140] = 0.25    # lower tiles
    v[140, 130, 256:] = 0.75
    g = vdbc.Grid(vdbc.encode(v, 1.0)[0])
    return g, torch.from_numpy(v).cuda(), g.background


def _positions(kind, dims):
    nx, ny, nz = dims
    if kind in ("lattice", "between"):   # rows along x, 7 short of a multiple of 64
        s = 0.0 if kind == "lattice" else 0.37
        z, y, x = np.meshgrid(np.arange(118, 136) + s, np.arange(115, 139) + s, np.arange(-1, nx) + s, indexing="ij")
        return np.stack([x, y, z], -1).reshape(-1, 3)
    if kind == "columns":                # along z: each lane in another row
        x, y, z = np.meshgrid(np.arange(120, 136) + 0.25, np.arange(120, 136) + 0.5, np.arange(-3, nz + 3) + 0.75,
                              indexing="ij")
        return np.stack([x, y, z], -1).reshape(-1, 3)
    t = np.linspace(0.0, 1.0, 30011)[:, None]
    if kind == "line":                   # some hundred positions a voxel
        return np.array([-3.0, 2.0, 1.0]) + t * np.array([nx + 5.0, ny - 1.0, nz + 2.0])
    if kind == "corner":                 # all lanes around one corner of eight leaves
        return np.array([127.5, 127.5, 127.5]) + 1.2 * (t - 0.5) * np.array([1.0, -1.0, 0.7])
    rng = np.random.default_rng(11)
    p = rng.uniform(-300.0, 500.0, (20011, 3))
    if kind == "faces":                  # just in and just out of the volume
        hi = np.array([nx, ny, nz], np.float64)
        p = np.where(rng.random((20011, 3)) < 0.5, rng.uniform(-2.5, 1.5, (20011, 3)), hi + rng.uniform(-2.5, 1.5, (20011, 3)))
        p = np.where(rng.random((20011, 3)) < 0.5, p, rng.uniform(0.0, 1.0, (20011, 3)) * hi)
    return p


@pytest.mark.parametrize("kind", ["lattice", "between", "columns", "line", "corner", "outside", "faces"])
def test_ordered_samples_equal_the_array_samples(scene, kind):
    g, dense, background = scene
    pos = torch.from_numpy(np.ascontiguousarray(_positions(kind, g.dims), np.float32)).cuda()
    want = vdbc.sample_dense(dense, background, pos, 1).view(torch.int32)
    for _ in range(8):
        assert torch.equal(vdbc.sample(g, pos, 1).view(torch.int32), want)
    assert want.unique().numel() > 50   # the positions are worth comparing
