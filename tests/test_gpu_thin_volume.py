"""A volume one voxel thick with 2^30 voxels in a plane: more macrocells than one
grid dimension of a launch takes threads for, and more rows of leaf regions than
a region index covers."""
import numpy as np
import pytest
import torch

from paper_2504_04564_amd import _build, vdbc
from synth import scenes

pytestmark = pytest.mark.gpu

NY, NZ = 32768, 32776


@pytest.fixture(scope="module")
def thin():
    _build.ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    vdbc.load()
    v = np.zeros((NZ, NY, 1), np.float32)
    rng = np.random.default_rng(4)
    for z, y in ((0, 0), (NZ - 90, NY - 77), (NZ // 2 - 40, 16384), (40, NY - 70), (NZ - 70, 33)):
        v[z:z + 70, y:y + 70] = rng.random(v[z:z + 70, y:y + 70].shape, dtype=np.float32)
    buf, st = vdbc.encode(v, 1e-4)
    # every voxel that is not background is stored: at most 9 bricks a patch
    assert st["k_bricks"] >= 45
    return vdbc.Grid(buf), torch.from_numpy(v).cuda()


@pytest.mark.parametrize("tree", [True, False])
def test_majorants_of_every_macrocell(thin, tree):
    g, dense = thin
    med = scenes.pt_medium(64.0)   # extinction = density: a cell's majorant is its footprint's largest value
    got = vdbc.majorant(g, med, 4) if tree else vdbc.majorant(dense, med, 4, 0.0)
    want = torch.nn.functional.max_pool2d(dense[None, None, :, :, 0], 6, 4, padding=1)[0, 0]
    want = want * torch.tensor(np.float32(64.0) / np.float32(NZ), device="cuda")
    assert got.shape == (NZ // 4, NY // 4, 1) and got.numel() * 64 >= 1 << 32
    assert torch.equal(got[..., 0], want)
