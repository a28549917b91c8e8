"""A streaming object alive while the context moves into a HIP stream under
capture and out of it again: the capture holds the draw made in it and nothing
else, its replays and the stream's records and totals are the oracle's."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W
from test_gpu_stream import _dev, _oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CHUNKS = [257, 256, 85, 1, 64]


@pytest.mark.parametrize("push_outside", [False, True])
def test_capture_beside_a_stream(push_outside):
    from paper_1805_08893_amd import vr
    m = W.icosphere_mesh(4, 4, "hilbert")
    sp = W.shader_for_mesh(m, W.SHADER_PHONG, 6, num_lights=2)
    rc, ora = vro.process_draw(m.indices, m.vertices, sp, vro.STATIC_HASH, 64)
    assert rc == vro.OK
    idx, vtx = _dev(m.indices), _dev(m.vertices)
    own, cap = torch.cuda.Stream(), torch.cuda.Stream()
    stage = vr.GeometryStage(0, stream=own)
    rec = torch.zeros((m.num_tris, 8), dtype=torch.float32, device="cuda")
    res = stage.alloc_outputs(m.num_tris, vr.VR_STATIC_HASH, 64, corners=True)
    torch.cuda.synchronize()
    st, h = vr.vr_stream_create(stage.ctx, 2, 257, 640, 480, rec)
    assert st == vr.VR_OK
    t0 = 0

    def push(n):
        nonlocal t0
        for T in CHUNKS[:n] if t0 == 0 else CHUNKS[-n:]:
            assert vr.vr_stream_push(h, idx[3 * t0:3 * (t0 + T)], vtx, sp, vr.VR_STATIC_HASH, 64) == vr.VR_OK
            t0 += T

    print(f"case push outside {push_outside}", flush=True)
    push(3)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=cap, capture_error_mode="thread_local"):
        assert vr.vr_set_stream(stage.ctx, cap) == vr.VR_OK
        assert vr.vr_process_draw_noalloc(stage.ctx, idx, vtx, sp, vr.VR_STATIC_HASH, 64, None,
                                          stage.describe(res)) == vr.VR_OK
        if push_outside:   # back on a stream of its own while the capture goes on
            assert vr.vr_set_stream(stage.ctx, own) == vr.VR_OK
            push(2)
    assert vr.vr_set_stream(stage.ctx, own) == vr.VR_OK
    for _ in range(3):
        res["corners"].zero_()
        res["counters"].fill_(3)
        g.replay()
        torch.cuda.synchronize()
        assert res["counters"].cpu().tolist() == [*ora["counters"][:2].tolist(), 0, 0]
        np.testing.assert_array_equal(res["corners"].cpu().numpy().view(np.uint32), ora["corners"].view(np.uint32))
    if not push_outside:
        push(2)
    st, tris, vis, inv = vr.vr_stream_finish(h)
    ref, rvis, rinv = _oracle(m, sp, CHUNKS, vro.STATIC_HASH, 64, 640, 480)
    assert st == vr.VR_OK and (tris, vis, inv) == (sum(CHUNKS), rvis, rinv)
    np.testing.assert_array_equal(rec[:tris].cpu().numpy().view(np.uint32), ref.view(np.uint32))
    vr.vr_stream_destroy(h)
    stage.close()
