"""The EA and ISO marchers with four lanes per ray (dense arrays, and VDBs read
through the region index) against the kernels with one thread per ray, which
the counting launches and the launches without an index still run: the same
arithmetic per sample in the same order, so the same bits.  Cameras near and
far, axis-parallel rays, images that do not fill their last tiles, every parity
of the bisection, early termination, and a transfer function that is not clear
at the background (nothing may be skipped then)."""
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


def _fields():
    cloud = synth.cloud_volume((61, 72, 90), seed=4)
    noise = np.random.default_rng(3).random((17, 31, 16), dtype=np.float32)
    return {"vdb": (vdbc.Grid(vdbc.encode(cloud, 0.15)[0]), None),
            "lossless": (vdbc.Grid(vdbc.encode(noise, 1.0)[0]), None),
            "nothing": (vdbc.Grid(vdbc.encode(np.zeros((9, 8, 7), np.float32), 0.5, flags=vdbc.NO_CORNERS)[0]), None),
            "dense": (torch.from_numpy(cloud).cuda(), 0.0)}


def _cameras(dims):
    nx, ny, nz = dims
    far = scenes.orbit_camera(dims, 23, 19, distance=400.0, fov_y_deg=0.3)
    side = dict(kind=0, width=19, height=9, lower_left=(nx + 3.0, -0.5, -0.5), du=(0.0, ny / 19, 0.0),
                dv=(0.0, 0.0, nz / 9), dir=(-1.0, 0.0, 0.0))
    return [scenes.orbit_camera(dims, 45, 35), scenes.ortho_z_camera(nx, ny, 8, 1), far, side]


def _both(field, cam, med, prm, mode, background, aov):
    a = vdbc.Renderer(field, cam, med, prm, mode, background=background, aov=aov)
    b = vdbc.Renderer(field, cam, med, dict(prm, flags=prm["flags"] | vdbc.RENDER_COUNT), mode, background=background,
                      aov=aov)
    a.image.fill_(-3.0)
    return a, _bits(a.launch()), b, _bits(b.launch())


@pytest.mark.parametrize("name", ["vdb", "lossless", "nothing", "dense"])
@pytest.mark.parametrize("flags", [0, vdbc.RENDER_HDDA])
def test_emission_absorption(name, flags):
    field, bg = _fields()[name]
    dims = field.dims if bg is None else tuple(reversed(field.shape))
    hazy = dict(scenes.ea_medium(6.0), tf=[(0.1, 0.2, 0.8, 0.05), (1.0, 0.9, 0.6, 1.0)])
    five = dict(scenes.ea_medium(20.0), tf=scenes.TF5, tf_range=scenes.TF5_RANGE)
    for cam in _cameras(dims):
        for med, step, t_end in ((scenes.ea_medium(8.0), 0.5, 0.0), (five, 0.37, 0.2), (hazy, 1.0, 0.0)):
            prm = dict(step=step, t_terminate=t_end, flags=flags)
            _, got, _, want = _both(field, cam, med, prm, vdbc.MODE_EA, bg, False)
            assert np.array_equal(got, want), (cam["kind"], step, t_end)


@pytest.mark.parametrize("name", ["vdb", "lossless", "nothing", "dense"])
@pytest.mark.parametrize("refine", [0, 1, 2, 7, 12])
def test_iso_surface(name, refine):
    field, bg = _fields()[name]
    dims = field.dims if bg is None else tuple(reversed(field.shape))
    for cam in _cameras(dims):
        for iso, step, flags in ((0.4, 0.5, vdbc.RENDER_HDDA), (0.0, 0.73, 0), (-0.5, 0.5, vdbc.RENDER_HDDA)):
            prm = dict(step=step, iso=iso, refine=refine, flags=flags)
            a, got, b, want = _both(field, cam, None, prm, vdbc.MODE_ISO, bg, True)
            assert np.array_equal(got, want), (cam["kind"], iso)
            assert np.array_equal(_bits(a.aov), _bits(b.aov)), (cam["kind"], iso)


def test_without_an_index_the_tree_is_marched_alike():
    g, _ = _fields()["vdb"]
    cam, med = scenes.orbit_camera(g.dims, 37, 21), scenes.ea_medium(8.0)
    r = vdbc.Renderer(g, cam, med, dict(step=0.5, flags=vdbc.RENDER_HDDA), vdbc.MODE_EA)
    want = _bits(r.launch()).copy()
    r.prm.flags &= ~vdbc.RENDER_INDEX
    assert np.array_equal(_bits(r.launch()), want)
    got = vdbc.render_noalloc(g, cam, med, dict(step=0.5, flags=vdbc.RENDER_INDEX), vdbc.MODE_EA)
    assert np.array_equal(_bits(got), want)
