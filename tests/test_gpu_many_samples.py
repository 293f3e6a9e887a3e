"""More samples in one call than a grid dimension takes threads."""
import numpy as np
import pytest
import torch

from paper_2504_04564_amd import _build, vdbc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("filter", [0, 1])
def test_every_sample_of_more_than_two_to_the_32(filter):
    _build.ensure_built()
    v = np.random.default_rng(1).random((20, 17, 33), dtype=np.float32)
    g = vdbc.Grid(vdbc.encode(v, 1.0, flags=vdbc.BG_EXPLICIT)[0])
    n = (1 << 32) + 1031
    if torch.cuda.mem_get_info()[0] < 18 * n:
        pytest.skip("needs 75 GB of device memory")
    pos = torch.zeros((n, 3), device="cuda")
    tail = torch.rand((5000, 3), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda") * 30.0
    pos[-5000:] = tail
    out = torch.full((n,), -1.0, device="cuda")
    for field, call in ((g, vdbc.sample), (torch.from_numpy(v).cuda(), lambda f, *a: vdbc.sample_dense(f, 0.0, *a))):
        out.fill_(-1.0)
        call(field, pos, filter, out)
        assert torch.equal(out[-5000:], call(field, tail, filter, torch.empty(5000, device="cuda")))
        assert float(out[: n - 5000].min()) == float(out[: n - 5000].max()) == float(v[0, 0, 0])
