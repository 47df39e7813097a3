"""Pruning where its tiles and chunks have edges: grids that do not fill their
last brick or group of bricks, one voxel, rows of all lengths, every pattern
of points a voxel, against the FP64 oracle; and the kept bits installed."""
import numpy as np
import pytest

from gpu_common import need_gpu, tiny_field
from oracle.pruning import grid_prune_fp64
from paper_2311_02542_amd import capi, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


@pytest.mark.parametrize("g,share", [(1, 1.0), (3, 0.5), (13, 0.2), (18, 1.0), (33, 0.03), (40, 0.4), (32, 0.0)])
@pytest.mark.parametrize("npts", [1, 4, 8, 27, 64])
def test_prune_edges(R, g, share, npts):
    torch = R.torch
    occ = np.random.default_rng(g).random((g, g, g)) < share
    if share == 0.0:
        occ[g - 1, 5, g - 1] = True
    f = tiny_field(g, occ, (-0.3, 0.1, 0.2), 1.5, seed=g, L=6, b_sigma=2.5)
    fid = R.load(f)
    words = (g ** 3 + 31) // 32
    bits = torch.full((words,), -1, dtype=torch.int32, device="cuda")
    mx = torch.zeros(g ** 3, device="cuda")
    capi.vrn_prune_grid(R.ctx, fid, 0.0, bits, mx, npts, "f32")
    assert np.array_equal(bits.cpu().numpy().view(np.uint32), synth.pack_bits(occ))      # alpha 0 keeps every voxel
    m = mx.cpu().numpy()
    assert np.array_equal(np.isnan(m), ~occ.ravel())
    alpha = float(np.median(m[occ.ravel()]))
    capi.vrn_prune_grid(R.ctx, fid, alpha, bits, None, npts, "f32")
    want, ref, tie = grid_prune_fp64(f, alpha, npts)
    # sigma is within 2e-6 relative (the FP32 MLP's bound): the opacity 1 - exp(-sigma dt) within 2e-6 / e
    assert np.nanmax(np.abs(m - ref)) < 1e-6
    got = synth.unpack_bits(bits.cpu().numpy().view(np.uint32), g).ravel()
    keep = synth.unpack_bits(want, g).ravel()
    assert np.array_equal(got[~tie], keep[~tie])
    R.unload(fid)
