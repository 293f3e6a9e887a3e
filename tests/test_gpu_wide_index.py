"""Region indexes that small volumes never need: entries in floats (a buffer past
4 GB) in the marchers and in a batch beside small volumes, and a batch in which
one volume has too many regions for an index.  Images are those of the tree
accessor bit for bit."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_04564_amd import _build, vdbc
from synth import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    _build.ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return vdbc.load()


@pytest.fixture(scope="module")
def wide():
    n = 1056   # 4.7 GB of values: leaves past 4 GB, an empty corner, constant regions
    x = np.arange(n, dtype=np.float32)
    v = np.empty((n, n, n), np.float32)
    for z in range(n):
        v[z] = ((x[:, None] * 3.0 + x[None, :] * 7.0 + z * 5.0) % 61.0) / 61.0
    v[:200, :150, :170] = 0.0
    v[512:560, 512:560, 512:560] = 0.5
    buf, _ = vdbc.encode(v, 1.0, flags=vdbc.BG_EXPLICIT)
    assert buf.size > 1 << 32
    return vdbc.Grid(buf)


def _small(seed):
    return vdbc.Grid(vdbc.encode(synth.cloud_volume((37, 50, 71), seed=seed), 0.25)[0])


def _bits(t):
    return t.view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("flags", [0, vdbc.RENDER_HDDA])
def test_marchers_with_wide_entries(wide, flags):
    dense_tf = dict(scenes.ea_medium(8.0), tf=[(0.1, 0.2, 0.8, 0.05), (1.0, 0.9, 0.6, 1.0)])   # nothing is skipped
    for az in (30.0, 220.0):
        cam = scenes.orbit_camera(wide.dims, 72, 53, azimuth_deg=az)
        for mode, med in ((vdbc.MODE_EA, scenes.ea_medium(8.0)), (vdbc.MODE_EA, dense_tf), (vdbc.MODE_ISO, None)):
            prm = dict(step=0.7, iso=0.4, refine=7)
            r = vdbc.Renderer(wide, cam, med, dict(prm, flags=flags), mode)
            every = vdbc.Renderer(wide, cam, med, dict(prm, flags=vdbc.RENDER_COUNT), mode)
            got = _bits(r.launch())
            assert np.array_equal(got, _bits(every.launch())), (az, mode)
            assert len(np.unique(got)) > 100


def _batch_equals_the_tree(grids, tuning):
    items, want = [], []
    for i, g in enumerate(grids):
        cam, med = scenes.orbit_camera(g.dims, 40 + i, 31, azimuth_deg=60.0 * i), scenes.pt_medium(32.0)
        items.append(dict(grid=g, camera=cam, medium=med, spp=3, max_bounces=4, seed=7 + i, frame=i))
        prm = dict(spp=3, max_bounces=4, seed=7 + i, frame=i, macrocell=tuning["macrocell"], flags=vdbc.RENDER_CACHE_LEAF)
        want.append(_bits(vdbc.render(g, cam, med, prm, vdbc.MODE_PT)))
    b = vdbc.Batch(items, tuning)
    for img in b.images:
        img.fill_(-1.0)
    b.launch()
    torch.cuda.synchronize()
    for i, (img, w) in enumerate(zip(b.images, want)):
        assert np.array_equal(_bits(img), w), i
    b.close()


@pytest.mark.parametrize("persistent", [1, 0])
def test_one_wide_volume_among_small_ones(wide, persistent):
    _batch_equals_the_tree([_small(3), wide, _small(4)], dict(macrocell=32, persistent=persistent, chunk_spp=2))


@pytest.mark.parametrize("persistent", [1, 0])
def test_one_volume_without_an_index(persistent):
    # 4098 x 4098 rows of regions and more are past what an index covers
    v = np.zeros((32768, 32768, 1), np.float32)
    v[16000:16800, 16000:16800] = np.random.default_rng(9).random((800, 800, 1), dtype=np.float32)
    thin = vdbc.Grid(vdbc.encode(v, 1e-3)[0])
    del v
    r = vdbc.Renderer(thin, scenes.orbit_camera(thin.dims, 16, 16), scenes.pt_medium(32.0), dict(macrocell=64),
                      vdbc.MODE_PT)
    without = vdbc.Renderer(thin, scenes.orbit_camera(thin.dims, 16, 16), scenes.pt_medium(32.0),
                            dict(macrocell=64, flags=vdbc.RENDER_CACHE_LEAF), vdbc.MODE_PT)
    assert r.ws_bytes == without.ws_bytes   # no bytes for an index
    _batch_equals_the_tree([_small(5), thin, _small(6)], dict(macrocell=64, persistent=persistent, chunk_spp=0))
