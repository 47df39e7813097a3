"""Host cameras of vrn_render, which go to the kernel with its arguments:
the same bits as device cameras for every number of cameras, each call its
own cameras without a wait between calls, and the caller's array free to
change at once; under graph capture the cameras are copied by the graph, so a
replay reads the (pinned) host memory anew."""
import ctypes

import pytest

from gpu_common import need_gpu
from paper_2311_02542_amd import capi, serve, synth

pytestmark = pytest.mark.gpu

W, H = 72, 40


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


def _render(R, fid, arr, n, out, compute, stream=None):
    opts = capi.render_opts(compute)
    rgba, ns = out
    handle = ctypes.c_void_p(stream.cuda_stream if stream else 0)
    st = capi.load_library().vrn_render(R.ctx, fid, arr, n, W, H, ctypes.byref(opts), rgba.data_ptr(), ns.data_ptr(),
                                        None, 0, handle)
    assert st == capi.VRN_OK


def _frames(R, n):
    torch = R.torch
    return torch.full((n, H, W, 4), -1.0, device="cuda"), torch.full((n, H, W), -1, dtype=torch.int32, device="cuda")


def _device(R, fid, cams, compute):
    torch = R.torch
    blob = bytes(capi.make_cameras(cams, H))
    d_cams = torch.frombuffer(bytearray(blob), dtype=torch.uint8).cuda()
    out = _frames(R, len(cams))
    capi.vrn_render_device_cams(R.ctx, fid, d_cams, len(cams), W, H, *out, compute)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("n", [1, 2, 15, 16])
@pytest.mark.parametrize("compute", ["f32", "f32x", "f16", "bf16"])
def test_host_cameras_equal_device_cameras(R, n, compute):
    torch = R.torch
    fid = R.load(synth.field_blobs64())
    cams = synth.cameras_blobs64(20, W, H)
    # three calls in a row, the array overwritten as soon as each returns
    arr = capi.make_cameras(cams[:n], H)
    outs = []
    for k in range(3):
        ctypes.memmove(arr, capi.make_cameras(cams[k:k + n], H), ctypes.sizeof(arr))
        outs.append(_frames(R, n))
        _render(R, fid, arr, n, outs[-1], compute)
        ctypes.memset(arr, 0xFF, ctypes.sizeof(arr))
    torch.cuda.synchronize()
    assert int(outs[0][1].sum()) > 0 and int(outs[1][1].sum()) > 0   # (one camera sees nothing)
    for k in range(3):
        want = _device(R, fid, cams[k:k + n], compute)
        assert torch.equal(outs[k][0], want[0]) and torch.equal(outs[k][1], want[1])
    R.unload(fid)


def test_captured_render_reads_the_host_cameras_at_replay(R):
    torch = R.torch
    fid = R.load(synth.field_blobs64())
    cams = synth.cameras_blobs64(4, W, H)
    pinned = torch.zeros(serve.CAM_BYTES, dtype=torch.uint8, pin_memory=True)
    arr = (capi.VrnCamera * 1).from_buffer(pinned.numpy())
    ctypes.memmove(arr, capi.make_cameras(cams[:1], H), ctypes.sizeof(arr))
    out = _frames(R, 1)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        _render(R, fid, arr, 1, out, "f16", stream)
    for cam in cams:
        ctypes.memmove(arr, capi.make_cameras([cam], H), ctypes.sizeof(arr))
        with torch.cuda.stream(stream):
            g.replay()
        stream.synchronize()
        want = _device(R, fid, [cam], "f16")
        assert torch.equal(out[0], want[0]) and torch.equal(out[1], want[1])
    R.unload(fid)
