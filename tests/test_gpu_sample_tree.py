"""Trilinear samples of a VDB, whose waves share the descents into the further
leaf regions of their footprints: equal bit for bit to the samples of the
reconstructed volume as a plain array (same interpolation of the same corners),
for every mix of crossed axes in a wave, ragged counts, constant regions and
positions outside the volume."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_04564_amd import _build, vdbc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scene():
    _build.ensure_built()
    v = synth.mid_volume(n=72)[:70, :61, :72].copy()
    v[8:24, 8:24, 8:24] = 0.25          # constant leaf regions
    g = vdbc.Grid(vdbc.encode(v, 0.4)[0])
    nx, ny, nz = g.dims
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    ijk = torch.from_numpy(np.stack([i, j, k], -1).reshape(-1, 3).astype(np.int32)).cuda()
    far = torch.tensor([[-2, -2, -2]], dtype=torch.int32, device="cuda")
    background = float(vdbc.lookup(g, far)[0])
    return g, vdbc.lookup(g, ijk).reshape(nz, ny, nx).contiguous(), background


def _positions(kind, n, dims, seed):
    rng = np.random.default_rng(seed)
    hi = np.array(dims, np.float32)
    p = rng.uniform(-3, hi + 2, (n, 3)).astype(np.float32)
    if kind == "all":        # every footprint reaches eight regions
        p = (8 * rng.integers(0, 8, (n, 3)) + 7 + rng.uniform(0, 0.999, (n, 3))).astype(np.float32)
    elif kind == "mixed":    # crossed axes at random, positions on the lattice too
        c = rng.integers(0, 2, (n, 3))
        p = (8 * rng.integers(-1, 9, (n, 3)) + np.where(c, 7, rng.integers(0, 7, (n, 3)))).astype(np.float32)
    elif kind == "tiles":
        p = rng.uniform(7, 25, (n, 3)).astype(np.float32)
    elif kind == "wild":
        p[::3] = [1e30, -np.inf, np.inf]
        p[1::5, 1] = np.nan
    return p


@pytest.mark.parametrize("kind", ["any", "all", "mixed", "tiles", "wild"])
@pytest.mark.parametrize("n", [1, 63, 65, 256, 1031])
def test_tree_samples_equal_the_array_samples(scene, kind, n):
    g, dense, background = scene
    pos = torch.from_numpy(_positions(kind, n, g.dims, n)).cuda()
    a, b = vdbc.sample(g, pos, 1), vdbc.sample_dense(dense, background, pos, 1)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
