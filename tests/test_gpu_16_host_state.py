"""What other code of the process has done with the HIP runtime: calls are not
refused for it."""
import ctypes

import pytest

from gpu_common import need_gpu
from paper_2311_02542_amd import capi, synth

pytestmark = pytest.mark.gpu
N = 40


@pytest.fixture(scope="module")
def R():
    need_gpu()
    r = capi.Renderer(0)
    yield r
    r.close()


def _hip():
    with open("/proc/self/maps") as maps:
        return ctypes.CDLL(sorted({line.split()[-1] for line in maps if "libamdhip64" in line})[0])


class NullStream:
    cuda_stream = 0


@pytest.mark.parametrize("mode", [1, 2])          # thread-local, relaxed
def test_host_cameras_on_the_null_stream_beside_a_capture(R, mode):
    torch, hip = R.torch, _hip()
    fid = R.load(synth.field_blobs64())
    cams = synth.cameras_blobs64(2, N, N)
    want = R.render(fid, cams, N, N, "f32")
    got = [torch.zeros_like(t) for t in want]
    stream, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0          # a blocking one
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(stream, mode) == 0
    try:
        for _ in range(2):
            capi.vrn_render(R.ctx, fid, cams, N, N, *got, "f32", workspace=R.ws, stream=NullStream)
    finally:
        ended = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
        hip.hipGetLastError()
    assert ended == 0
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and int(want[1].sum()) > 0
    assert hip.hipGraphDestroy(graph) == 0 and hip.hipStreamDestroy(stream) == 0
    R.unload(fid)


def test_load_after_another_call_has_failed(R):
    R.torch.cuda.synchronize()
    assert _hip().hipSetDevice(1 << 20) != 0          # leaves its error as the thread's last one
    fid = R.load(synth.field_blobs64())
    _hip().hipGetLastError()
    cams = synth.cameras_blobs64(1, N, N)
    assert int(R.render(fid, cams, N, N, "f32")[1].sum()) > 0
    R.unload(fid)
