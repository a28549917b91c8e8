"""The buffers a destroyed stream leaves to its context serve the next stream
and are given back when no stream needs them any more."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_buffers_are_kept_and_given_back():
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    rec = torch.zeros((1 << 20, 8), dtype=torch.float32, device="cuda")

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    def stream():
        st, h = vr.vr_stream_create(stage.ctx, 1, 1 << 20, 640, 480, rec)   # 144 MiB
        assert st == vr.VR_OK
        vr.vr_stream_destroy(h)

    assert stage.sync()[0] == vr.VR_OK
    before, size = free(), 144 << 20
    stream()
    kept = free()
    assert before - kept >= size
    for _ in range(3):   # a sync between streams that follow each other keeps them
        assert stage.sync()[0] == vr.VR_OK
        stream()
        assert free() == kept
    assert stage.sync()[0] == vr.VR_OK and stage.sync()[0] == vr.VR_OK
    assert free() >= before
    stream()
    assert before - free() >= size
    stage.close()
    assert free() >= before
