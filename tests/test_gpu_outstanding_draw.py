"""A draw of few batches still running on one HIP stream while the context, by
then on another, synchronises or searches candidates: the draw's counters, and
those of the draws that use its arrival word afterwards, against the oracle."""
import time

import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

WORDS = 64   # arrival words of a context, taken in turn


@pytest.mark.parametrize("meanwhile", ["sync", "autotune"])
def test_counters_of_a_draw_outstanding_on_another_stream(meanwhile):
    from paper_1805_08893_amd import vr
    from paper_1805_08893_amd.autotune import vr_autotune
    # four long batches of a dear vertex program and one of a single triangle, which arrives at once
    whole = W.grid_mesh(64, 64, 3, "random")
    ind = whole.indices[:3 * (4 * 1024 + 1)].copy()
    sp = W.shader_for_mesh(whole, W.SHADER_OFFSET, 3, iterations=4096)
    rc, ora = vro.process_draw(ind, whole.vertices, sp, vro.STATIC_BALLOT, 1024)
    assert rc == vro.OK
    small = ind[:3 * 100].copy()
    cheap = W.shader_for_mesh(whole, W.SHADER_MVP, 3)
    rc, so = vro.process_draw(small, whole.vertices, cheap, vro.STATIC_HASH, 16)
    assert rc == vro.OK
    idx, sidx = (torch.from_numpy(a.view(np.int32)).cuda() for a in (ind, small))
    vtx = torch.from_numpy(whole.vertices).cuda()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    stage = vr.GeometryStage(0, stream=a)
    res = stage.alloc_outputs(len(ind) // 3, vr.VR_STATIC_BALLOT, 1024, corners=True)
    sres = [stage.alloc_outputs(100, vr.VR_STATIC_HASH, 16, corners=True) for _ in range(WORDS)]
    ended = torch.cuda.Event()
    torch.cuda.synchronize()
    print(f"case {meanwhile}", flush=True)
    stage.draw(idx, vtx, sp, vr.VR_STATIC_BALLOT, 1024, res=res)
    ended.record(a)
    assert vr.vr_set_stream(stage.ctx, b) == vr.VR_OK
    time.sleep(0.001)
    outstanding = not ended.query()
    if meanwhile == "sync":
        assert stage.sync()[0] == vr.VR_OK
    else:
        vr_autotune(stage.ctx, sidx, vtx, cheap, [(vr.VR_STATIC_HASH, 16, 0)], 1)
    torch.cuda.synchronize()
    assert outstanding, "the draw ended too early to show anything"
    assert res["counters"].cpu().tolist() == [*ora["counters"][:2].tolist(), 0, 0]
    np.testing.assert_array_equal(res["corners"].cpu().numpy().view(np.uint32), ora["corners"].view(np.uint32))
    for r in sres:
        stage.draw(sidx, vtx, cheap, vr.VR_STATIC_HASH, 16, res=r)
    torch.cuda.synchronize()
    for r in sres:
        assert r["counters"].cpu().tolist() == [*so["counters"][:2].tolist(), 0, 0]
    assert stage.sync()[0] == vr.VR_OK
    stage.close()
