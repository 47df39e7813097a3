"""Pruning passes and occupancy installs of one field from several streams:
each waits for the one before it, so each gives what it gives alone; a captured
pass waits for nothing and replays."""
import numpy as np
import pytest

from gpu_common import need_gpu, tiny_field
from paper_2311_02542_amd import capi, synth

pytestmark = pytest.mark.gpu
G = 128


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


def _field(seed):
    occ = np.random.default_rng(seed).random((G, G, G)) < 0.3
    return tiny_field(G, occ, (-0.3, 0.1, 0.2), 1.5, seed=3, L=6, b_sigma=2.5)


def _prune(R, fid, alpha, bits, opacity, compute, stream=None):
    capi.vrn_prune_grid(R.ctx, fid, alpha, bits, opacity, 4, compute, stream=stream)


def _outputs(R):
    torch = R.torch
    return torch.zeros(G ** 3 // 32, dtype=torch.int32, device="cuda"), torch.zeros(G ** 3, device="cuda")


def test_overlapping_calls_of_one_field(R):
    torch = R.torch
    f, other = _field(1), _field(2)
    grids = [torch.from_numpy(g["occ_bits"].view(np.int32)).cuda() for g in (f, other)]
    fid = R.load(f)
    bits, opacity = _outputs(R)
    _prune(R, fid, 0.0, bits, opacity, "f16")
    seen = opacity[~torch.isnan(opacity)]
    alphas = [float(torch.quantile(seen[::7], q)) for q in (0.1, 0.5, 0.9)]

    def passes(streams):
        """Three passes on the first grid, the install of the second, three passes on it and the first again."""
        out = []
        for k, grid in enumerate(grids):
            for i, alpha in enumerate(alphas):
                out.append(_outputs(R))
                torch.cuda.synchronize()
                for _ in range(3):
                    _prune(R, fid, alpha, *out[-1], "f16", streams[i])
                    _prune(R, fid, alphas[0], bits, None, "f16", streams[(i + 1) % 3])
            capi.vrn_set_occupancy(R.ctx, fid, grids[1 - k], stream=streams[(k + 1) % 3])
        out.append(R.render(fid, synth.cameras_blobs64(1, 64, 64), 64, 64, "f16", stream=streams[2]))
        torch.cuda.synchronize()
        return out

    alone = passes([torch.cuda.current_stream()] * 3)
    for _ in range(3):
        for a, b in zip(alone, passes([torch.cuda.Stream() for _ in range(3)])):
            assert torch.equal(a[0], b[0]) and torch.equal(torch.nan_to_num(a[1], -1.0), torch.nan_to_num(b[1], -1.0))
    R.unload(fid)


def test_captured_pass_replays(R):
    torch = R.torch
    fid = R.load(_field(1))
    want, got = _outputs(R), _outputs(R)
    _prune(R, fid, 0.3, *want, "f32")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        _prune(R, fid, 0.3, *got, "f32", stream)
    for _ in range(3):
        got[0].zero_()
        got[1].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(want[0], got[0])
        assert torch.equal(torch.nan_to_num(want[1], -1.0), torch.nan_to_num(got[1], -1.0))
        _prune(R, fid, 0.3, *want, "f32")
        torch.cuda.synchronize()
    R.unload(fid)
