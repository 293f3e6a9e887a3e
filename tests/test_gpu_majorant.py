"""Majorant grids at every split of the work: macrocells of a wave (up to 16)
and of a workgroup, edges that are no multiple of a leaf, and dense runs of 64,
128 and 256 columns with their ragged ends, against the oracle (float64: a few
roundings of the transfer function's lookup and of the product) and, tree
against its reconstruction, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_04564_amd import _build, vdbc

pytestmark = pytest.mark.gpu

MED = dict(sigma_scale=6.0, tf=[(0.2, 0.3, 0.9, 0.0), (0.9, 0.1, 0.2, 0.8), (0.4, 0.4, 0.4, 0.3),
                                (1.0, 1.0, 0.0, 1.0), (0.0, 1.0, 1.0, 0.5)], tf_range=(0.1, 0.9))


@pytest.fixture(scope="module", autouse=True)
def lib():
    _build.ensure_built()
    return vdbc.load()


def _volume(nx, ny, nz, seed):
    rng = np.random.default_rng(seed)
    v = rng.random((nz, ny, nx)).astype(np.float32)
    v[rng.random((nz, ny, nx)) < 0.6] = 0.0
    v[:, :, : nx // 3] *= 0.2          # cells of different ranges
    return v


@pytest.mark.parametrize("nx", [1, 64, 65, 128, 129, 256, 300])
@pytest.mark.parametrize("C", [4, 5, 15, 16, 17, 31, 48, 63, 64])
def test_majorants_at_the_edges_of_their_splits(nx, C):
    v = _volume(nx, 19, 35, nx + C)
    buf, st = vdbc.encode(v, 0.4)
    got = vdbc.majorant(vdbc.Grid(buf), MED, C).cpu().numpy()
    np.testing.assert_allclose(got, oracle.majorant(oracle.VdbField(buf), MED, C), rtol=2e-6, atol=1e-12)
    for field in (v, oracle.reconstruct(v, 0.4)):
        dense = vdbc.majorant(torch.from_numpy(np.ascontiguousarray(field)).cuda(), MED, C,
                              background=st["background"]).cpu().numpy()
        want = oracle.majorant(oracle.DenseField(field, st["background"]), MED, C)
        np.testing.assert_allclose(dense, want, rtol=2e-6, atol=1e-12)
    assert np.array_equal(got.view(np.uint32), dense.view(np.uint32))
