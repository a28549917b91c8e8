"""Draws of few batches end without a reduction launch: counters, totals and
look-back words at one batch, at the most such a draw has (128), one more and
in between, twice in a row with every output, on every batched strategy, with
draws of both kinds in turn and on two HIP streams, against the oracle."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("strategy,bt,nu", [(vro.STATIC_HASH, 8, 0), (vro.STATIC_SORT, 8, 0), (vro.STATIC_BALLOT, 8, 0),
                                            (vro.DYN_HASH, 8, 9), (vro.DYN_SORT, 8, 9), (vro.DYN_PHASH, 8, 9),
                                            (vro.DYN_BALLOT, 8, 9)])
def test_counters_around_the_limit(strategy, bt, nu):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    whole = W.grid_mesh(40, 37, 4, "hilbert")
    sp = W.shader_for_mesh(whole, W.SHADER_MVP, 4)
    vtx = torch.from_numpy(whole.vertices).cuda()
    torch.cuda.synchronize()
    turn = 0
    for T in (1, 8, 9, 127 * 3, 128 * 3, 127 * 8, 128 * 8, 128 * 8 + 1, 130 * 8):
        ind = whole.indices[:3 * T].copy()
        print(f"case {strategy} T={T}", flush=True)
        rc, ora = vro.process_draw(ind, whole.vertices, sp, strategy, bt, {"max_unique": nu})
        assert rc == 0
        inv, units = int(ora["counters"][0]), int(ora["counters"][1])
        idx = torch.from_numpy(ind.view(np.int32)).cuda()
        torch.cuda.synchronize()
        for every in (True, True, False):
            vr.vr_set_stream(stage.ctx, streams[turn % 2])
            turn += 1
            res = stage.draw(idx, vtx, sp, strategy, bt, dict(max_unique=nu), corners=True, tris=every, verts=every,
                             units=every)
            torch.cuda.synchronize()
            assert res["counters"].cpu().tolist() == [inv, units, 0, 0]
            np.testing.assert_array_equal(res["corners"].cpu().numpy().view(np.uint32), ora["corners"].view(np.uint32))
            if every:
                np.testing.assert_array_equal(res["tris"].cpu().numpy().view(np.uint32), ora["tris"])
        st, total = stage.sync()
        assert st == vr.VR_OK and total == 3 * inv
    stage.close()
