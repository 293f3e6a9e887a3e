"""Calls at the limits of the marchers with four lanes per ray, against the
kernels with one thread per ray (counting launches): cameras so far away that a
position's rounding passes the skips' margin, a termination threshold that
ends a ray at its first sample, and images with more lanes than one grid
dimension takes."""
import math

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


def _bits(t):
    return t.view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("voxels", [8.0e3, 2.0e4, 3.2e4, 3.0e5, 1.0e6])
def test_skipping_is_exact_from_far_away(voxels):
    # asked for or not, empty blocks change nothing: the image of every sample
    n = 256
    g = vdbc.Grid(vdbc.encode(synth.mid_volume(n=n), 0.10)[0])
    fov = math.degrees(2.0 * math.atan(0.6 * n / voxels))
    for az in (10.0, 75.0, 200.0):
        cam = scenes.orbit_camera(g.dims, 320, 320, fov_y_deg=fov, azimuth_deg=az, distance=voxels / n)
        for mode, med in ((vdbc.MODE_EA, scenes.ea_medium(8.0)), (vdbc.MODE_ISO, None)):
            every = vdbc.Renderer(g, cam, med, dict(step=0.5, iso=0.3, flags=vdbc.RENDER_COUNT), mode)
            want = _bits(every.launch())
            for flags in (0, vdbc.RENDER_HDDA):
                r = vdbc.Renderer(g, cam, med, dict(step=0.5, iso=0.3, flags=flags), mode)
                assert np.array_equal(_bits(r.launch()), want), (az, mode, flags)


@pytest.mark.parametrize("flags", [0, vdbc.RENDER_HDDA])
@pytest.mark.parametrize("t_end", [1.0, 1.5])
@pytest.mark.parametrize("dense", [False, True])
def test_termination_at_the_first_sample(dense, t_end, flags):
    vol = synth.cloud_volume((61, 72, 90), seed=4)
    dims = tuple(reversed(vol.shape))
    field, bg = (torch.from_numpy(vol).cuda(), 0.0) if dense else (vdbc.Grid(vdbc.encode(vol, 0.15)[0]), None)
    cam, med = scenes.orbit_camera(dims, 70, 50), scenes.ea_medium(8.0)
    prm = dict(step=0.5, t_terminate=t_end, flags=flags)
    r = vdbc.Renderer(field, cam, med, prm, vdbc.MODE_EA, background=bg)
    every = vdbc.Renderer(field, cam, med, dict(prm, flags=flags | vdbc.RENDER_COUNT), vdbc.MODE_EA, background=bg)
    assert np.array_equal(_bits(r.launch()), _bits(every.launch()))


def test_images_past_two_to_the_thirty_pixels():
    # 4 lanes a pixel: 2^32 + 2^20 threads
    w, h = 32768, 32776
    vol = np.random.default_rng(2).random((3, 16, 16), dtype=np.float32)
    g = vdbc.Grid(vdbc.encode(vol, 1.0, flags=vdbc.BG_EXPLICIT)[0])
    cam = dict(kind=0, width=w, height=h, lower_left=(-1.0, -1.0, -1.0), du=(18.0 / w, 0.0, 0.0),
               dv=(0.0, 18.0 / h, 0.0), dir=(0.0, 0.0, 1.0))
    dense = torch.from_numpy(vol).cuda()
    for field, mode, bg in ((g, vdbc.MODE_EA, None), (dense, vdbc.MODE_ISO, 0.0)):
        med, prm = scenes.ea_medium(8.0), dict(step=1.0, iso=0.5, refine=1)
        r = vdbc.Renderer(field, cam, med, prm, mode, background=bg)
        every = vdbc.Renderer(field, cam, med, dict(prm, flags=vdbc.RENDER_COUNT), mode, background=bg)
        r.image.fill_(-1.0)
        r.launch()
        every.launch()
        assert float(r.image[-2000, w // 2, 3]) >= 0.0
        for y in range(0, h, 4096):
            a, b = r.image[y:y + 4096], every.image[y:y + 4096]
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), y
        del r, every
        torch.cuda.empty_cache()


@pytest.mark.parametrize("distance", [0.8, 2.5])
@pytest.mark.parametrize("flags", [0, vdbc.RENDER_HDDA])
def test_long_volumes(distance, flags):
    # a side of 20000: within and past what may be skipped by the region index
    v = np.zeros((20000, 24, 31), np.float32)
    rng = np.random.default_rng(8)
    for z in (0, 3000, 9991, 19970):
        v[z:z + 30] = rng.random((30, 24, 31), dtype=np.float32)
    g = vdbc.Grid(vdbc.encode(v, 0.05)[0])
    cam = scenes.orbit_camera(g.dims, 90, 60, azimuth_deg=3.0, elevation_deg=1.0, distance=distance,
                              fov_y_deg=0.2)
    for mode, med in ((vdbc.MODE_EA, scenes.ea_medium(8000.0)), (vdbc.MODE_ISO, None)):
        prm = dict(step=0.5, iso=0.5, refine=5)
        r = vdbc.Renderer(g, cam, med, dict(prm, flags=flags), mode)
        every = vdbc.Renderer(g, cam, med, dict(prm, flags=flags | vdbc.RENDER_COUNT), mode)
        got = _bits(r.launch())
        assert np.array_equal(got, _bits(every.launch())), mode
        assert len(np.unique(got)) > 20, mode
