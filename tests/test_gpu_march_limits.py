"""Calls at the limits of the marchers with four lanes per ray, against the
kernels with one thread per ray (counting launches): cameras so far away that a
position's rounding passes the skips' margin, and a termination threshold that
ends a ray at its first sample."""
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


@pytest.mark.parametrize("voxels", [3.0e5, 1.0e6])
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
