"""Triangle setup inside the draw kernels of a stream: chunks at the edges of
the naive workgroup (85 triangles), of a batch and of a wavefront's triangles,
two streams alive at once, a stream in the buffers an earlier one left, and
pushes before and after the context moves to another HIP stream; records and
totals bitwise against the oracle."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W
from test_gpu_stream import _dev, _oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CHUNKS = [1, 63, 64, 65, 84, 85, 86, 170, 171, 255, 256, 257]


def _scene():
    m = W.icosphere_mesh(4, 4, "hilbert", swap_frac=0.05)
    return m, W.shader_for_mesh(m, W.SHADER_PHONG, 6, num_lights=2)


def _push(vr, stage, h, idx, vtx, sp, gs, bt, chunks, t0=0):
    for T in chunks:
        assert vr.vr_stream_push(h, idx[3 * t0:3 * (t0 + T)], vtx, sp, gs, bt) == vr.VR_OK, vr.vr_last_error(stage.ctx)
        t0 += T
    return t0


def _check(vr, h, rec, m, sp, chunks, name, bt):
    st, tris, vis, inv = vr.vr_stream_finish(h)
    ref, rvis, rinv = _oracle(m, sp, chunks, vro.STRATEGY_NAMES.index(name), bt, 640, 480)
    assert st == vr.VR_OK and (tris, vis, inv) == (sum(chunks), rvis, rinv)
    np.testing.assert_array_equal(rec[:tris].cpu().numpy().view(np.uint32), ref.view(np.uint32))
    return rinv


@pytest.mark.parametrize("name,bt", [("naive", 1), ("static_ballot", 64), ("static_ballot", 7), ("static_hash", 21),
                                     ("static_hash", 85), ("static_hash", 256), ("static_sort", 21),
                                     ("static_sort", 64), ("static_sort", 256)])
def test_chunk_edges(name, bt):
    from paper_1805_08893_amd import vr
    m, sp = _scene()
    stage = vr.GeometryStage(0)
    idx, vtx = _dev(m.indices), _dev(m.vertices)
    print(f"[stream units] {name} {bt}", flush=True)
    total = 0
    for slots in (1, 3):   # the second stream takes the first one's buffers or larger ones
        rec = torch.zeros((m.num_tris, 8), dtype=torch.float32, device="cuda")
        st, h = vr.vr_stream_create(stage.ctx, slots, 257, 640, 480, rec)
        assert st == vr.VR_OK
        _push(vr, stage, h, idx, vtx, sp, vr.STRATEGIES[name], bt, CHUNKS)
        total += _check(vr, h, rec, m, sp, CHUNKS, name, bt)
        vr.vr_stream_destroy(h)
    st, inv = stage.sync()
    assert st == vr.VR_OK and inv == total   # the context's total counts streams too
    stage.close()


def test_two_streams_and_another_hip_stream():
    from paper_1805_08893_amd import vr
    m, sp = _scene()
    stage = vr.GeometryStage(0)
    idx, vtx = _dev(m.indices), _dev(m.vertices)
    recs = [torch.zeros((m.num_tris, 8), dtype=torch.float32, device="cuda") for _ in range(2)]
    hs = [vr.vr_stream_create(stage.ctx, 2, 257, 640, 480, r)[1] for r in recs]
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    gs, half = vr.VR_STATIC_HASH, len(CHUNKS) // 2
    at = [_push(vr, stage, h, idx, vtx, sp, gs, 64, CHUNKS[:half]) for h in hs]
    assert vr.vr_set_stream(stage.ctx, other) == vr.VR_OK
    for h, t in zip(hs, at):
        _push(vr, stage, h, idx, vtx, sp, gs, 64, CHUNKS[half:], t)
    for h, r in zip(hs, recs):
        _check(vr, h, r, m, sp, CHUNKS, "static_hash", 64)
        vr.vr_stream_destroy(h)
    stage.close()
