"""The library's own choice of samples per work item (RENDER_SPLIT with
chunk_spp 0): images and AOVs are those of whole tiles bit for bit, a workspace
without room for the pixel sums renders whole tiles, and the workspace grows
only where the tiles are split."""
import ctypes as C

import pytest
import torch

import synth
from paper_2504_04564_amd import _build, vdbc
from synth import scenes


def _bytes(w, h, spp, flags=vdbc.RENDER_SPLIT, tw=8, camera=True):
    prm = vdbc.params_c(dict(spp=spp, flags=flags, tile_w=tw), vdbc.MODE_PT)
    cam = vdbc.camera_c(dict(kind=0, width=w, height=h, dir=(0, 0, 1)))
    ws = C.c_uint64(0)
    st = vdbc.load().vdbc_render_workspace(C.byref(prm), vdbc.Dims(16, 16, 16), C.byref(cam) if camera else None,
                                           C.byref(ws))
    return st, ws.value


def test_workspace_of_the_library_split():
    _build.ensure_built()
    base = _bytes(64, 64, 4, flags=0)[1]
    # one sample is never split; two are in a small image
    assert _bytes(64, 64, 1) == (vdbc.OK, base)
    assert _bytes(64, 64, 1, tw=128)[0] == vdbc.E_INVALID
    assert _bytes(64, 64, 1, tw=128, flags=0) == (vdbc.OK, base)   # refused by the render
    assert _bytes(64, 64, 2) == (vdbc.OK, base + 40 * 64 * 64)
    assert _bytes(64, 64, 2, tw=128)[0] == vdbc.E_INVALID
    assert _bytes(64, 64, 2, camera=False)[0] == vdbc.E_INVALID
    # 6143 tiles of 32 x 8 are split, 6144 are not; more than 1280 work items
    # are queued in cost order, also where one sample leaves nothing to split
    order = lambda tiles: -(-(512 + 8 * tiles) // 256) * 256
    sums = lambda pixels: -(-40 * pixels // 256) * 256
    assert _bytes(32 * 6143, 8, 4) == (vdbc.OK, base + sums(32 * 6143 * 8) + order(6143))
    assert _bytes(32 * 6144, 8, 4) == (vdbc.OK, base + order(6144))
    assert _bytes(32 * 1280, 8, 1) == (vdbc.OK, base)
    assert _bytes(32 * 1281, 8, 1) == (vdbc.OK, base + order(1281))
    assert _bytes(32 * 320, 8, 4) == (vdbc.OK, base + sums(32 * 320 * 8))
    assert _bytes(32 * 321, 8, 4) == (vdbc.OK, base + sums(32 * 321 * 8) + order(321))
    # thin volumes past 2^24 index rows have no index
    prm = vdbc.params_c(dict(spp=1, flags=vdbc.RENDER_INDEX), vdbc.MODE_EA)
    ws = C.c_uint64(0)
    for rows, some in ((4096, True), (8 * 4095, False)):
        assert vdbc.load().vdbc_render_workspace(C.byref(prm), vdbc.Dims(8, 8 * 4095, rows), None, C.byref(ws)) == 0
        assert (ws.value > 0) == some


@pytest.mark.gpu
@pytest.mark.parametrize("w,h,spp,dense", [(70, 33, 13, False), (33, 70, 2, True), (512, 200, 3, False), (520, 470, 4, False),
                                            (1300, 512, 1, False)])
def test_split_by_the_library_is_bit_identical(w, h, spp, dense):
    _build.ensure_built()
    v = synth.mid_volume(n=64)
    field = torch.from_numpy(v).cuda() if dense else vdbc.Grid(vdbc.encode(v, 0.25)[0])
    cam, med = scenes.orbit_camera((64, 64, 64), w, h), scenes.pt_medium(64.0)
    prm = dict(spp=spp, max_bounces=8, seed=3, macrocell=8)
    bg = 0.0 if dense else None
    r = vdbc.Renderer(field, cam, med, prm, vdbc.MODE_PT, aov=True, background=bg)
    assert r.prm.flags & vdbc.RENDER_SPLIT
    r.ws.fill_(0xA5)
    a = r.launch().clone(), r.aov.clone()
    whole = vdbc.Renderer(field, cam, med, dict(prm, chunk_spp=spp), vdbc.MODE_PT, aov=True, background=bg)
    assert not whole.prm.flags & vdbc.RENDER_SPLIT and whole.ws_bytes <= r.ws_bytes
    b = whole.launch().clone(), whole.aov.clone()
    assert all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))
    # no room for the sums and the order: whole tiles
    r.ws_bytes = whole.ws_bytes
    r.image.zero_()
    assert torch.equal(r.launch().view(torch.int32), b[0].view(torch.int32))
    r.ws_bytes = whole.ws_bytes - 1
    with pytest.raises(vdbc.VdbcError):
        r.launch()
