"""Render launches whose blocks hold waves that only help to copy the weights:
frames at the changes in how many waves of a block carry rays (one a block up
to 256 x 16 rays, eight at 256 x 8 x 16) give the bits of the same cameras in
a batch that fills the chip, and two such launches at once on two streams do
not disturb each other."""
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


# 8x8 tiles: 1, 64, 65 (two carrying waves a block), 193 and 256 (four: all
# of a 16-bit block), 257, 448 and 449 (seven and eight), 512, 513
@pytest.mark.parametrize("tiles", [1, 64, 65, 193, 256, 257, 448, 449, 512, 513])
@pytest.mark.parametrize("compute", ["f32", "f32x", "f16", "bf16"])
def test_frames_of_few_waves_a_block(R, tiles, compute):
    torch = R.torch
    fid = R.load(synth.field_blobs64())
    W, H = 8 * tiles, 8
    cams = synth.cameras_blobs64(8, W, H)
    want, want_n = R.render(fid, cams * 2, W, H, compute)
    torch.cuda.synchronize()
    before = R.stats()["rays"]
    got, got_n = R.render(fid, cams[:1], W, H, compute)
    torch.cuda.synchronize()
    assert R.stats()["rays"] - before == W * H
    assert torch.equal(got[0], want[0]) and torch.equal(got_n[0], want_n[0])
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    ws = [torch.zeros(capi.vrn_workspace_bytes(R.ctx), dtype=torch.uint8, device="cuda") for _ in streams]
    out = [torch.full((1, H, W, 4), -1.0, device="cuda") for _ in streams]
    torch.cuda.synchronize()
    for k, s in enumerate(streams):
        capi.vrn_workspace_init(R.ctx, ws[k], stream=s)
        for _ in range(3):
            capi.vrn_render(R.ctx, fid, cams[k + 1:k + 2], W, H, out[k], None, compute, workspace=ws[k], stream=s)
    torch.cuda.synchronize()
    for k in range(2):
        assert torch.equal(out[k][0], want[k + 1])
    R.unload(fid)
