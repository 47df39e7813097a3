"""Launch shapes of the render kernel: frames of sizes around the changes in
how many rays a wave carries (16, 32, 64) and how rays are dealt to waves and
queues give the same bits as the same cameras rendered in one large batch or
in row bands, write every pixel once and count every ray."""
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


def _render(R, fid, cams, W, H, compute):
    torch = R.torch
    rgba = torch.full((len(cams), H, W, 4), float("nan"), device="cuda")
    ns = torch.full((len(cams), H, W), -1, dtype=torch.int32, device="cuda")
    before = R.stats()["rays"]
    R.render(fid, cams, W, H, compute, out=(rgba, ns))
    torch.cuda.synchronize()
    return rgba, ns, R.stats()["rays"] - before


# 256 CUs hold 4096 waves: 16 rays a wave up to 65,536 rays (256 x 256), 32 up
# to 131,072; one tile, one wave, one block; 7 and 8 queues' worth of blocks
@pytest.mark.parametrize("W,H", [(1, 1), (8, 8), (17, 9), (56, 8), (64, 8), (65, 33), (256, 256), (264, 256),
                                 (362, 360), (368, 368), (520, 505), (801, 640)])
@pytest.mark.parametrize("compute", ["f32", "f16"])
def test_launch_shapes_agree(R, W, H, compute):
    torch = R.torch
    fid = R.load(synth.field_blobs64())
    cams = synth.cameras_blobs64(4, W, H)
    want, want_n, rays = _render(R, fid, cams * 4, W, H, compute)
    assert rays == 16 * W * H
    rgba, ns, rays = _render(R, fid, cams[:1], W, H, compute)
    assert rays == W * H and bool((ns >= 0).all()) and not bool(rgba.isnan().any())
    assert torch.equal(rgba[0], want[0]) and torch.equal(ns[0], want_n[0])
    assert torch.equal(want[4:8], want[:4]) and torch.equal(want_n[12:], want_n[:4])
    if H > 1:
        cut = H // 3 + 1
        parts = [dict(cams[1], row_begin=0, row_end=cut), dict(cams[1], row_begin=cut, row_end=H)]
        rgba, ns, rays = _render(R, fid, parts, W, H, compute)
        assert rays == W * H
        both = torch.cat([rgba[0, :cut], rgba[1, cut:]])
        assert torch.equal(both, want[1]) and bool((ns[0, cut:] == -1).all()) and bool((ns[1, :cut] == -1).all())
    R.unload(fid)
