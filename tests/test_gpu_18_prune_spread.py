"""Pruning over counts and spreads of voxels: chunks from one voxel to sixteen,
and tiles with one to sixteen points of a voxel side by side.  A voxel's
opacity has the same bits whatever voxels stand beside it."""
import numpy as np
import pytest

from gpu_common import need_gpu, tiny_field
from paper_2311_02542_amd import capi, synth

pytestmark = pytest.mark.gpu
G = 64


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


def _grids():
    """Scattered voxels, from one to more than a turn of full chunks for every wave; then rows, planes across
    each axis and blocks: runs along x of one voxel and more."""
    rng = np.random.default_rng(5)
    order = rng.permutation(G ** 3)
    for n in (1, 2, 7, 300, 6000, 11000, 17000, 30000, 60000, 100000):
        occ = np.zeros(G ** 3, bool)
        occ[order[:n]] = True
        yield occ.reshape(G, G, G)
    for axis in range(3):
        occ = np.zeros((G, G, G), bool)
        occ[tuple(slice(None) if a != axis else slice(1, None, 5) for a in range(3))] = True
        yield occ
    occ = np.zeros((G, G, G), bool)
    occ[10:13, 20:41, 3:9] = True
    occ[11, 30, 5] = False
    yield occ


@pytest.mark.parametrize("npts", [1, 4, 8, 27, 64])
@pytest.mark.parametrize("compute", ["f32", "f16", "bf16", "f32x"])
def test_opacity_does_not_depend_on_other_voxels(R, npts, compute):
    torch = R.torch
    fid = R.load(tiny_field(G, np.ones((G, G, G), bool), (-0.3, 0.1, 0.2), 1.5, seed=9, L=9, b_sigma=2.5,
                            table_dtype=np.float16 if compute == "f16" else np.float32))
    bits = torch.zeros(G ** 3 // 32, dtype=torch.int32, device="cuda")
    full, some = torch.zeros(G ** 3, device="cuda"), torch.zeros(G ** 3, device="cuda")
    capi.vrn_prune_grid(R.ctx, fid, 0.0, bits, full, npts, compute)
    alpha = float(full[::5].median())
    for k, occ in enumerate(_grids()):
        held = torch.from_numpy(synth.pack_bits(occ).view(np.int32)).cuda()
        capi.vrn_set_occupancy(R.ctx, fid, held)
        capi.vrn_prune_grid(R.ctx, fid, alpha, bits, some, npts, compute)
        want = torch.where(torch.from_numpy(occ.ravel()).cuda(), full, torch.nan)
        assert torch.equal(torch.nan_to_num(some, -1.0), torch.nan_to_num(want, -1.0)), f"grid {k}"
        kept = synth.unpack_bits(bits.cpu().numpy().view(np.uint32), G).ravel()
        assert np.array_equal(kept, occ.ravel() & (full.cpu().numpy() >= np.float32(alpha))), f"grid {k}"
    torch.cuda.synchronize()
    R.unload(fid)
