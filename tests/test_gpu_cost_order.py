"""Cost order of the path tracer's tiles: fewer and more tiles than the sorting
workgroup has threads, a single tile, and a medium that gives every tile the
same cost; each order holds every tile once, so the image is that of raster
order bit for bit."""
import pytest
import torch

import synth
from paper_2504_04564_amd import _build, vdbc
from synth import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,tw", [(8, 8, 8), (300, 1100, 8), (64, 1024, 64), (33, 1025, 64)])
@pytest.mark.parametrize("sigma", [64.0, 0.0])
def test_order_holds_every_tile_once(w, h, tw, sigma):
    _build.ensure_built()
    g = vdbc.Grid(vdbc.encode(synth.mid_volume(n=64), 0.25)[0])
    cam, med = scenes.orbit_camera((64, 64, 64), w, h), dict(scenes.pt_medium(64.0), sigma_scale=sigma)
    prm = dict(spp=1, max_bounces=4, seed=9, macrocell=8, tile_w=tw)
    a = vdbc.Renderer(g, cam, med, prm, vdbc.MODE_PT).launch()
    r = vdbc.Renderer(g, cam, med, dict(prm, flags=vdbc.RENDER_COST_ORDER), vdbc.MODE_PT)
    r.ws.fill_(0xA5)
    r.image.fill_(-1.0)
    b = r.launch()
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    # the order itself, after the bins
    tiles = ((w + 4 * tw - 1) // (4 * tw)) * ((h + 64 // tw - 1) // (64 // tw))
    vol = 256 + (-(-4 * 8 ** 3 // 256)) * 256 + 256          # counters, 8^3 majorants, one coarse block's bits
    at = r.ws_off + vol + 512 + 4 * tiles
    order = r.ws[at:at + 4 * tiles].view(torch.int32)
    assert torch.equal(order.sort().values.cpu(), torch.arange(tiles, dtype=torch.int32))
