"""Convolution paths of the denoiser that its own layers do not take: stride-2 data gradients whose
weights do not fit in LDS beside the window, part-filled epilogue passes, and
the rounding of BF16 outputs at its edges."""
import numpy as np
import pytest
import torch

from oracle import nn
from paper_2504_04564_amd import _build, vdbc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    _build.ensure_built()
    return vdbc.load()


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _bf(rng, shape, scale=1.0):
    t = torch.from_numpy(rng.normal(size=shape).astype(np.float32) * np.float32(scale)).to(torch.bfloat16)
    return t.cuda(), t.to(torch.float64).numpy()


@pytest.mark.parametrize("cin,stride,cout,hs,ws", [
    (64, 1, 16, 11, 37), (32, 1, 56, 9, 33), (64, 2, 64, 18, 70), (16, 2, 64, 17, 33), (32, 2, 40, 8, 64),
])
def test_forward_and_data_gradient(cin, stride, cout, hs, ws):
    rng = np.random.default_rng(cin + cout + hs)
    a, a64 = _bf(rng, (1, hs, ws, cin))
    w, w64 = _bf(rng, (cout, 3, 3, cin), 0.2)
    bias = torch.zeros(cout, device="cuda")
    ref = nn.conv_fwd(a64, w64, np.zeros(cout), stride)
    got = vdbc.conv3x3(a, None, 0, stride, w, bias, cout, relu=False)
    assert rel(got.float().cpu().numpy(), ref) <= 4e-3          # one BF16 rounding: 2^-8 at most
    got = vdbc.conv3x3(a, None, 0, stride, w, bias, cout, relu=False, out_f32=True)
    assert rel(got.cpu().numpy(), ref) <= 1e-5
    dz, dz64 = _bf(rng, ref.shape[:3] + (cout,))     # cout is a multiple of 8 in these cases
    dx = vdbc.conv3x3_dgrad(dz, cout, w, cin, stride, hs, ws).cpu().numpy()
    assert rel(dx, nn.conv_dgrad(dz64, w64, a64.shape, stride)) <= 1e-5


def test_bf16_outputs_round_to_nearest_even():
    # all weights zero: the output is the bias, rounded
    bits = np.array([0x00000000, 0x80000000, 0x3F808000, 0x3F818000, 0x3F807FFF, 0x3F808001, 0xBF818000, 0x7F7FFFFF,
                     0x7F800000, 0xFF800000, 0x7FC00000, 0x00800000, 0x7F7F7FFF, 0x33333333, 0xC2C8C000, 0x3EAAAAAB],
                    np.uint32)
    bias = torch.from_numpy(bits.view(np.float32).copy()).cuda()
    a = torch.ones((1, 8, 32, 32), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((16, 3, 3, 32), dtype=torch.bfloat16, device="cuda")
    got = vdbc.conv3x3(a, None, 0, 1, w, bias, 16, relu=False)
    want = (bias + 0.0).to(torch.bfloat16).expand(1, 8, 32, 16)
    ok = (got.view(torch.int16) == want.contiguous().view(torch.int16)) | (got.isnan() & want.isnan())
    assert bool(ok.all()), (got[0, 0, 0], want[0, 0, 0])


@pytest.mark.parametrize("h,w", [(730, 722), (1030, 1026)])
def test_stride_two_forward_of_large_images(h, w):
    # more pixel tiles a wave from 131,072 and 262,144 output pixels on: the
    # rows are those of a strip of the image, bit for bit
    gen = torch.Generator(device="cuda").manual_seed(h)
    a = torch.randn((1, h, w, 32), generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn((64, 3, 3, 32), generator=gen, device="cuda").to(torch.bfloat16)
    bias = torch.randn(64, generator=gen, device="cuda")
    out = vdbc.conv3x3(a, None, 0, 2, k, bias, 64, relu=True)
    for y in (0, (h // 2) & ~1, (h - 48) & ~1):
        strip = vdbc.conv3x3(a[:, y:y + 48].contiguous(), None, 0, 2, k, bias, 64, relu=True)
        lo = 0 if y == 0 else 1
        assert torch.equal(out[:, y // 2 + lo:y // 2 + 23], strip[:, lo:23])
