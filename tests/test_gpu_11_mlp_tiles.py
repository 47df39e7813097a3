"""The MLP stage kernel where its tiles, waves and resident blocks have edges:
a sample's result has the same bits whatever stands beside it, and no value
beyond the last sample is written."""
import numpy as np
import pytest

from gpu_common import need_gpu
from paper_2311_02542_amd import capi, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


# one tile and its edges; the change from 4 to more waves a block (256 CUs);
# more tiles than resident waves, so that waves take a second and a third
@pytest.mark.parametrize("n", [1, 15, 16, 17, 4 * 256 * 16 + 1, 8 * 256 * 16 + 7, 3 * 32 * 256 * 16 - 5])
@pytest.mark.parametrize("compute", ["f32", "f16", "bf16", "f32x"])
@pytest.mark.parametrize("levels", [8, 16])
def test_results_do_not_depend_on_the_launch(R, n, compute, levels):
    torch = R.torch
    f = synth.field_blobs64() if levels == 8 else synth.field_room256(log2_T=4)
    fid = R.load(f)
    g = torch.Generator("cuda").manual_seed(n)
    x = torch.randn((n, 2 * levels), generator=g, device="cuda") * 0.1
    d = torch.nn.functional.normalize(torch.randn((n, 3), generator=g, device="cuda"), dim=1)
    sigma, rgb = torch.full((n + 64,), -7.0, device="cuda"), torch.full((n + 64, 3), -7.0, device="cuda")
    odd = torch.cat([x.new_zeros(1), x.flatten()])[1:]      # features that start between 8-byte boundaries
    assert odd.data_ptr() % 8 == 4
    capi.vrn_mlp(R.ctx, fid, odd, d, n, compute, sigma, rgb)
    assert bool((sigma[n:] == -7).all()) and bool((rgb[n:] == -7).all()) and bool((sigma[:n] > 0).all())
    at = torch.unique(torch.cat([torch.arange(min(n, 40)), torch.arange(max(0, n - 40), n),
                                 torch.from_numpy(np.random.default_rng(n).integers(0, n, 200))])).cuda()
    s2, c2 = torch.empty(at.numel(), device="cuda"), torch.empty((at.numel(), 3), device="cuda")
    capi.vrn_mlp(R.ctx, fid, x[at].contiguous(), d[at].contiguous(), at.numel(), compute, s2, c2)
    assert torch.equal(s2, sigma[at]) and torch.equal(c2, rgb[at])
    R.unload(fid)
