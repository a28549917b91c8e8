"""Draws of few batches with a plan that was not made for them: one of smaller
budgets (more batches than the draw's bound), one of a longer stream, an empty
one.  The batches within the bound are drawn and counted, and the draws that
follow, which take every arrival word of the context again, count as always."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

WORDS = 64   # arrival words of a context, taken in turn


def _counts(ind, vtx, sp, starts, ballot):
    """Invocations and units of the batches [starts[i], starts[i + 1])."""
    s, bt = (vro.STATIC_BALLOT, 1024) if ballot else (vro.STATIC_HASH, 256)
    rows = [vro.process_draw(ind[3 * a:3 * b], vtx, sp, s, bt)[1]["counters"][:2] for a, b in zip(starts, starts[1:])]
    return [int(x) for x in np.sum(rows, axis=0)] if rows else [0, 0]


# strategy, N_pmax, N_u, triangles drawn and planned, the plan's budgets, the draw's batch bound; whether every batch is drawn
CASES = [("dyn_hash", 64, 256, 100, 100, (30, 256), 2, False),
         ("dyn_phash", 64, 256, 129, 129, (8, 256), 3, False),
         ("dyn_sort", 341, 64, 300, 300, (8, 64), 15, True),     # grid-stride: batches past the bound are drawn too
         ("dyn_ballot", 85, 64, 300, 300, (8, 64), 15, False),
         ("dyn_ballot", 64, 256, 100, 100, (2, 256), 2, False),
         ("dyn_hash", 64, 256, 100, 400, (64, 256), 2, True),    # a longer stream of full batches
         ("dyn_hash", 64, 256, 100, 0, None, 2, False)]


@pytest.mark.parametrize("name,bt,nu,T,planned,budgets,bound,whole", CASES)
def test_counters_and_later_draws(name, bt, nu, T, planned, budgets, bound, whole):
    from paper_1805_08893_amd import vr
    m = W.grid_mesh(21, 17, 4, "hilbert")
    sp = W.shader_for_mesh(m, W.SHADER_MVP, 4)
    ind = m.indices[:3 * T].copy()
    starts = [] if budgets is None else vro.plan_dynamic(m.indices[:3 * planned], len(m.vertices), budgets[1], budgets[0]).tolist()
    assert bound == T // min(bt, (nu - 2 + 2) // 3) + 1 and (not starts or len(starts) - 1 > bound)
    plan = np.zeros(max(planned, T) + 2, np.int32)
    plan[0] = max(0, len(starts) - 1)
    plan[1:1 + len(starts)] = starts
    mine = [min(s, T) for s in starts[:bound + 1]]
    _, ref = vro.process_draw(ind, m.vertices, sp, vro.NAIVE, 1)
    _, ora = vro.process_draw(ind, m.vertices, sp, vro.STRATEGY_NAMES.index(name), bt, {"max_unique": nu})
    idx, vtx, dplan = torch.from_numpy(ind.view(np.int32)).cuda(), torch.from_numpy(m.vertices).cuda(), torch.from_numpy(plan).cuda()
    stage = vr.GeometryStage(0)
    gs = vr.STRATEGIES[name]
    print(f"case {name} {bt}/{nu} T={T} plan of {plan[0]}", flush=True)
    res = stage.alloc_outputs(T, gs, bt, corners=True)
    res["counters"].fill_(7)
    stage.draw(idx, vtx, sp, gs, bt, dict(max_unique=nu, plan=dplan), res=res)
    assert stage.sync()[0] == vr.VR_OK
    assert res["counters"].cpu().tolist() == [*_counts(ind, m.vertices, sp, mine, name == "dyn_ballot"), 0, 0]
    drawn = 3 * (T if whole else mine[-1] if mine else 0)
    np.testing.assert_array_equal(res["corners"].cpu().numpy()[:drawn].view(np.uint32), ref["corners"][:drawn].view(np.uint32))
    for _ in range(WORDS):
        r = stage.draw(idx, vtx, sp, gs, bt, dict(max_unique=nu), corners=True)
        torch.cuda.synchronize()
        assert r["counters"].cpu().tolist() == [*ora["counters"][:2].tolist(), 0, 0]
    assert stage.sync()[0] == vr.VR_OK
    stage.close()


def test_batches_past_the_bound_leave_no_trace():
    """More batches than the allocation-free draw's array holds: every triangle
    is drawn, the batches within the bound are counted, and the look-back words
    behind the array's aggregates are as they were."""
    from paper_1805_08893_amd import vr
    T = 524288 + 1000   # the array holds 524,288 batches
    m = W.grid_mesh(513, 520, 4, "scan")
    sp = W.shader_for_mesh(m, W.SHADER_MVP, 4)
    idx, vtx = torch.from_numpy(m.indices[:3 * T].view(np.int32)).cuda(), torch.from_numpy(m.vertices).cuda()
    plan = torch.cat([torch.tensor([T]), torch.arange(T + 1)]).to(torch.int32).cuda()
    stage = vr.GeometryStage(0)
    bound = T // 85 + 1
    print(f"case T={T} bound {bound}", flush=True)
    naive = stage.draw(idx, vtx, sp, vr.VR_NAIVE, 1, corners=True)
    res = stage.alloc_outputs(T, vr.VR_DYN_HASH, 341, corners=True)
    opts = vr.make_opts(max_unique=256, plan=plan)
    assert vr.vr_process_draw_noalloc(stage.ctx, idx, vtx, sp, vr.VR_DYN_HASH, 341, opts, stage.describe(res)) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    assert res["counters"].cpu().tolist() == [3 * bound, bound, 0, 0]
    assert torch.equal(res["corners"].view(torch.int32), naive["corners"].view(torch.int32))
    n = 3000
    rc, ora = vro.process_draw(m.indices[:3 * n], m.vertices, sp, vro.STATIC_HASH, 1)
    assert rc == vro.OK
    res = stage.alloc_outputs(n, vr.VR_STATIC_HASH, 1, corners=True, tris=True, verts=True, units=True)
    assert vr.vr_process_draw_noalloc(stage.ctx, idx[:3 * n], vtx, sp, vr.VR_STATIC_HASH, 1, None, stage.describe(res)) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    np.testing.assert_array_equal(res["tris"].cpu().numpy().view(np.uint32), ora["tris"])
    np.testing.assert_array_equal(res["unit_invocations"].cpu().numpy().view(np.uint32)[:n], ora["unit_invocations"])
    stage.close()
