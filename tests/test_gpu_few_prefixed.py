"""Indexed draws around the most batches that clear their own look-back words
(32), one after another on the same words, and in turn with draws that leave
the clearing to the reduction: every draw's outputs against the oracle."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("name,bt", [("static_hash", 8), ("static_sort", 8), ("static_ballot", 8)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_repeated_prefixed_draws(name, bt, noalloc):
    from paper_1805_08893_amd import vr
    m = W.grid_mesh(30, 31, 4, "hilbert")
    sp = W.shader_for_mesh(m, W.SHADER_MVP, 4)
    vtx = torch.from_numpy(m.vertices).cuda()
    gs = vr.STRATEGIES[name]
    stage = vr.GeometryStage(0)
    draws = []
    for T in (1, 31 * bt, 32 * bt, 32 * bt + 1, 40 * bt):
        ind = m.indices[:3 * T].copy()
        rc, ora = vro.process_draw(ind, m.vertices, sp, vro.STRATEGY_NAMES.index(name), bt)
        assert rc == vro.OK
        res = [stage.alloc_outputs(T, gs, bt, corners=True, tris=True, verts=True, units=True) for _ in range(8)]
        draws.append((torch.from_numpy(ind.view(np.int32)).cuda(), res, ora))
    print(f"case {name} noalloc {noalloc}", flush=True)
    call = vr.vr_process_draw_noalloc if noalloc else vr.vr_process_draw
    for k in range(8):   # nothing waits between the draws
        for idx, res, _ in draws:
            assert call(stage.ctx, idx, vtx, sp, gs, bt, None, stage.describe(res[k])) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    for idx, res, ora in draws:
        inv, units = (int(x) for x in ora["counters"][:2])
        for r in res:
            assert r["counters"].cpu().tolist() == [inv, units, 0, 0]
            np.testing.assert_array_equal(r["tris"].cpu().numpy().view(np.uint32), ora["tris"])
            np.testing.assert_array_equal(r["verts"].cpu().numpy()[:inv].view(np.uint32), ora["verts"].view(np.uint32))
            np.testing.assert_array_equal(r["unit_offsets"].cpu().numpy().view(np.uint32)[:units + 1], ora["unit_offsets"])
    stage.close()
