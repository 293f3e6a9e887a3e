"""Stride-2 forward convolutions with one, two and four pixel tiles a wave, chosen
by input channels and output pixels: the rows of a large image are those of a
strip of it, which takes the smallest launch, bit for bit."""
import pytest
import torch

from paper_2504_04564_amd import _build, vdbc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin", [8, 24, 32, 48, 56, 64])
@pytest.mark.parametrize("h,w", [(330, 346), (512, 514), (730, 722), (1030, 1026)])
def test_large_images_equal_their_strips(cin, h, w):
    _build.ensure_built()
    gen = torch.Generator(device="cuda").manual_seed(h + cin)
    a = torch.randn((1, h, w, cin), generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn((40 if cin == 24 else 64, 3, 3, cin), generator=gen, device="cuda").to(torch.bfloat16)
    cout = k.shape[0]
    bias = torch.randn(cout, generator=gen, device="cuda")
    out = vdbc.conv3x3(a, None, 0, 2, k, bias, cout, relu=True)
    for y in (0, (h // 2) & ~1, (h - 14) & ~1):
        strip = vdbc.conv3x3(a[:, y:y + 14, :300].contiguous(), None, 0, 2, k, bias, cout, relu=True)
        lo = 0 if y == 0 else 1
        assert torch.equal(out[:, y // 2 + lo:y // 2 + 6, :149], strip[:, lo:6, :149])
