"""The serving engine's choice of a slot: with the shapes' buffers captured
ahead on every slot, a request goes to a slot that has a free buffer, so
held results cost no new capture before every slot's buffer is held, however
soon each request ends."""
import pytest

from gpu_common import need_gpu
from paper_2311_02542_amd import serve, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_slots", [1, 2, 3])
def test_held_results_use_the_other_slots_buffers(n_slots):
    torch = need_gpu()
    srv = serve.Server({"A": synth.field_blobs64()}, 1 << 30, n_slots=n_slots, compute="f16", use_graphs=True)
    srv.warmup([(256, 256, 1)])
    n0 = srv.stats()["captures"]
    assert n0 == n_slots
    srv.start()
    held = []
    for k in range(n_slots + 1):
        r = srv.submit("A", *synth.request_cameras("A", "preview", 70 + k))
        assert r.done.wait(60) and r.error is None
        held.append(r)
        assert srv.stats()["captures"] == (n0 if k < n_slots else n0 + 1)
    # every held result is a buffer of its own
    assert len({r.result[0].data_ptr() for r in held}) == n_slots + 1
    first = held[0].result[0].clone()
    held.pop().release()
    # and the released one is free for the next request
    r = srv.submit("A", *synth.request_cameras("A", "preview", 70))
    assert r.done.wait(60) and r.error is None
    torch.cuda.synchronize()
    assert srv.stats()["captures"] == n0 + 1
    assert torch.equal(r.result[0], first)
    for q in held + [r]:
        q.release()
    srv.stop(drain=True)
    srv.close()
