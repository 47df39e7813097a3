"""Rays along the planes of the grid -- directions with components of exactly
+0 or -0, eyes on cell and brick planes and one FP32 value beside them, eyes so
far that a position's error is a good part of a cell: their evaluated samples
equal the dense-masked march, and they take no more lattice tests than the
rays beside them."""
import itertools

import numpy as np
import pytest

from gpu_common import axis_camera, need_gpu
from oracle.march import dense_masked_march
from oracle.rays import canonical_rays
from paper_2311_02542_amd import capi, synth
from test_gpu_7_distance_skips import _field

pytestmark = pytest.mark.gpu
N = 9                  # odd, with cx = cy = N / 2: the middle row and column have components of exactly 0
# signed axes, the columns (right, down, forward), each forward both ways; the last gives zeros of both signs
AXES = [np.array(m, float) for m in ([[1, 0, 0], [0, 1, 0], [0, 0, 1]], [[0, 0, 1], [1, 0, 0], [0, 1, 0]],
                                     [[0, 1, 0], [0, 0, 1], [1, 0, 0]], [[0, 0, -1], [0, 1, 0], [1, 0, 0]],
                                     [[-1, 0, 0], [0, 0, -1], [0, -1, 0]],
                                     [[-1, -0.0, -0.0], [-0.0, 1, -0.0], [-0.0, -0.0, -1]])]


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


def _mid(f, kind):
    return np.array([0.3, -0.2, 0.1]) if kind == "contracted" else np.asarray(f["aabb_min"], float) + 0.5 * f["extent"]


def _eyes(f, kind):
    """Eyes on cell and brick planes, beside them and between them."""
    cell = float(f["extent"]) / f["occ_res"] * (f["radius"] if kind == "contracted" else 1.0)
    lo = _mid(f, kind) - 0.5 * f["occ_res"] * cell
    at = np.floor(0.5 * f["occ_res"] + np.array([0.0, 1.0, -1.0]))
    plane = (lo + cell * at).astype(np.float32)
    brick = (lo + cell * (at - at % 4)).astype(np.float32)
    return [plane, brick, np.nextafter(plane, np.float32(-9)), np.nextafter(brick, np.float32(9)),
            (lo + cell * (at + 0.4)).astype(np.float32)]


@pytest.mark.parametrize("kind,g", [("bounded", 61), ("bounded", 128), ("table", 30), ("contracted", 64)])
def test_samples_bit_exact(R, kind, g):
    torch = R.torch
    f = _field(kind, g)
    fid = R.load(f)
    jj, ii = np.meshgrid(np.arange(N), np.arange(N), indexing="ij")
    mk = 4096
    kl = torch.zeros((len(AXES) * N * N, mk), dtype=torch.int32, device="cuda")
    cnt = torch.zeros(len(AXES) * N * N, dtype=torch.int32, device="cuda")
    for e, eye in enumerate(_eyes(f, kind)):
        # half of the views from outside, against their direction of view
        cams = [axis_camera(m, eye - (e % 2) * 1.3 * f["extent"] * m[:, 2], N, N, fx=30.0, cx=N / 2, cy=N / 2) for m in AXES]
        capi.vrn_march(R.ctx, fid, cams, N, N, kl, mk, cnt)
        for i, cam in enumerate(cams):
            o, d = canonical_rays(cam, ii.ravel(), jj.ravel())
            assert (d == 0).sum() == 2 * N and bool((np.signbit(d) & (d == 0)).any()) == (i == 5)
            ks, want = dense_masked_march(f, o, d)
            at = slice(i * N * N, (i + 1) * N * N)
            np.testing.assert_array_equal(cnt[at].cpu().numpy(), want, err_msg=f"eye {e} camera {i}")
            m = int(want.max(initial=0))
            live = np.arange(m)[None, :] < want[:, None]
            got = kl[at, :max(m, 1)].cpu().numpy()[:, :m]
            np.testing.assert_array_equal(np.where(live, got, -1), np.where(live, ks[:, :m], -1),
                                          err_msg=f"eye {e} camera {i}")
    R.unload(fid)


def _corners(g):
    """Only one cell in from the corners of the grid is occupied: wide empty boxes."""
    occ = np.zeros((g, g, g), bool)
    for corner in itertools.product((1, g - 2), repeat=3):
        occ[corner] = True
    return synth.pack_bits(occ)


def _tests(R, fid, cam, rows):
    """Lattice tests of some rows of one view."""
    capi.vrn_workspace_init(R.ctx, R.ws)
    R.render(fid, [dict(cam, row_begin=rows[0], row_end=rows[1])], N, N, "f32")
    return R.stats()["march_steps"]


@pytest.mark.parametrize("kind", ["bounded", "table", "contracted"])
def test_no_more_lattice_tests_than_beside(R, kind):
    f = dict(_field(kind, 128), occ_bits=_corners(128))
    fid = R.load(f)
    for e, eye in enumerate(_eyes(f, kind)):
        for i, m in enumerate(AXES):
            cam = axis_camera(m, eye, N, N, fx=30.0, cx=N / 2, cy=N / 2)
            beside = max(_tests(R, fid, cam, (N // 2 - 1, N // 2)), _tests(R, fid, cam, (N // 2 + 1, N // 2 + 2)))
            # a ray along a plane crosses no more empty boxes than one that leaves it; a test more at each end
            assert _tests(R, fid, cam, (N // 2, N // 2 + 1)) <= beside + 2 * N, f"eye {e} camera {i}"
    R.unload(fid)


def test_far_eye(R):
    # an eye 1000 grids away: the bound on a position's error, delta, is a quarter of a cell
    torch = R.torch
    f = dict(_field("bounded", 128), occ_bits=_corners(128))
    fid = R.load(f)
    out = 1000.0 * f["extent"]
    mid = _mid(f, "bounded")
    # through the occupied cells of two corners of the grid, and beside them
    cams = [axis_camera(m, mid - out * m[:, 2] + f["extent"] * 63 / 128 * np.ones(3) * (1 - np.abs(m[:, 2])), N, N,
                        fx=1e6, cx=N / 2, cy=N / 2) for m in AXES]
    cnt = torch.zeros(len(AXES) * N * N, dtype=torch.int32, device="cuda")
    capi.vrn_march(R.ctx, fid, cams, N, N, torch.zeros((cnt.numel(), 1), dtype=torch.int32, device="cuda"), 1, cnt)
    jj, ii = np.meshgrid(np.arange(N), np.arange(N), indexing="ij")
    seen = 0
    for i, cam in enumerate(cams):
        _, want = dense_masked_march(f, *canonical_rays(cam, ii.ravel(), jj.ravel()))
        np.testing.assert_array_equal(cnt[i * N * N:(i + 1) * N * N].cpu().numpy(), want, err_msg=f"camera {i}")
        seen += int(want.sum())
    assert seen > 0
    capi.vrn_workspace_init(R.ctx, R.ws)
    R.render(fid, cams, N, N, "f32")
    # 423 samples of a ray lie in the grid; a skip spans most of it, and leaves the samples of the two cells
    # before a box's end and of the two corner cells
    s = R.stats()
    assert s["march_steps"] < 100 * s["rays"]
    R.unload(fid)
