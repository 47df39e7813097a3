"""FP32 products on the BF16 matrix cores: features whose neighbours differ by
many binary orders (every residual of the three-part split is then of its own
size, in both places of a pair) give results as close to FP64 as the FP32
matrix cores do."""
import numpy as np
import pytest

from gpu_common import need_gpu
from oracle.mlp import color_mlp, density_mlp
from oracle.sh import sh_basis
from paper_2311_02542_amd import capi, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


@pytest.mark.parametrize("low", [0, -12, -60, -140])
@pytest.mark.parametrize("n", [1, 16, 4099])
def test_split_products_as_exact_as_fp32(R, low, n):
    torch = R.torch
    f = synth.field_room256(log2_T=4)
    rng = np.random.default_rng(n - low)
    x = (rng.choice([-1, 1], (n, 32)) * rng.uniform(0.5, 1.0, (n, 32))
         * 2.0 ** rng.integers(low, 1, (n, 32))).astype(np.float32)
    d = rng.normal(size=(n, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    sigma, geo = density_mlp(x, f["mlp"])
    rgb = color_mlp(geo, sh_basis(d.astype(np.float64), 4), f["mlp"])
    fid = R.load(f)
    err = {}
    for compute in ("f32", "f32x"):
        s, c = torch.empty(n, device="cuda"), torch.empty((n, 3), device="cuda")
        capi.vrn_mlp(R.ctx, fid, torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda(), n, compute, s, c)
        err[compute] = (np.abs(s.cpu().numpy() / sigma - 1).max(), np.abs(c.cpu().numpy() - rgb).max())
    R.unload(fid)
    # both round FP32 sums in different orders, of some 32 to 64 products a unit:
    # twice the other's error, or the bounds the FP32 paths are held to
    assert err["f32x"][0] <= max(2 * err["f32"][0], 2e-6), err
    assert err["f32x"][1] <= max(2 * err["f32"][1], 1e-6), err
