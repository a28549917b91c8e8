"""Draws and frames whose units take the device's LDS to the last bytes: sizes
that the counted LDS allows, with the kernel's arrangement larger than counted
(a dynamic sort with its table) and equal to the limit, against the oracle; a
frame whose tables leave no room for the kernel's own 16 bytes is refused."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mesh():
    m = W.grid_mesh(131, 127, 4, "random")
    return m, W.shader_for_mesh(m, W.SHADER_MVP, 4)


@pytest.mark.parametrize("strategy,bt,nu,corners", [("dyn_sort", 2721, 4093, False), ("dyn_sort", 2721, 4096, False),
                                                    ("dyn_sort", 1041, 3029, True), ("dyn_hash", 1038, 3029, True)])
@pytest.mark.parametrize("wg", [0, 512])
def test_draw(mesh, strategy, bt, nu, corners, wg):
    from paper_1805_08893_amd import vr
    m, sp = mesh
    rc, ora = vro.process_draw(m.indices, m.vertices, sp, vro.STRATEGY_NAMES.index(strategy), bt, {"max_unique": nu})
    assert rc == vro.OK
    stage = vr.GeometryStage(0)
    gs = vr.STRATEGIES[strategy]
    idx, vtx = torch.from_numpy(m.indices.view(np.int32)).cuda(), torch.from_numpy(m.vertices).cuda()
    print(f"case {strategy} {bt}/{nu} corners {corners} wg {wg}", flush=True)
    res = stage.draw(idx, vtx, sp, gs, bt, dict(max_unique=nu, wg_size=wg), corners=corners, tris=True, verts=True)
    assert stage.sync()[0] == vr.VR_OK, vr.vr_last_error(stage.ctx)
    inv, units = (int(x) for x in ora["counters"][:2])
    assert res["counters"].cpu().tolist() == [inv, units, 0, 0]
    np.testing.assert_array_equal(res["tris"].cpu().numpy().view(np.uint32), ora["tris"])
    np.testing.assert_array_equal(res["verts"].cpu().numpy()[:inv].view(np.uint32), ora["verts"].view(np.uint32))
    if corners:
        np.testing.assert_array_equal(res["corners"].cpu().numpy().view(np.uint32), ora["corners"].view(np.uint32))
    stage.close()


# bytes of LDS: 163,824, 163,820 and 163,832
@pytest.mark.parametrize("strategy,bt,nu,draws,fits", [("dyn_hash", 1089, 3023, 3, True), ("dyn_hash", 1011, 3027, 66, True),
                                                       ("dyn_hash", 1038, 3029, 1, False)])
def test_frame(mesh, strategy, bt, nu, draws, fits):
    from paper_1805_08893_amd import vr
    m, sp = mesh
    n = 1500   # triangles a draw
    stage = vr.GeometryStage(0)
    gs, os_ = vr.STRATEGIES[strategy], vro.STRATEGY_NAMES.index(strategy)
    vtx = torch.from_numpy(m.vertices).cuda()
    idx, plans, outs, cnts, entries = [], [], [], [], []
    for d in range(draws):
        part = m.indices[3 * 8 * d:3 * (8 * d + n)].copy()
        idx.append(torch.from_numpy(part.view(np.int32)).cuda())
        plans.append(torch.zeros(n + 2, dtype=torch.int32, device="cuda"))
        assert vr.vr_plan_dynamic(stage.ctx, idx[d], len(m.vertices), nu, bt, plans[d]) == vr.VR_OK
        outs.append(torch.zeros((3 * n, 12), dtype=torch.float32, device="cuda"))
        cnts.append(torch.zeros(4, dtype=torch.int64, device="cuda"))
        entries.append(vr.make_draw(idx[d], vtx, 0, gs, bt, outs[d], cnts[d], nu, plans[d]))
    print(f"case frame {strategy} {bt}/{nu} of {draws}", flush=True)
    st = vr.vr_process_draws(stage.ctx, entries, [sp])
    assert st == (vr.VR_OK if fits else vr.VR_ERR_ARG), vr.vr_last_error(stage.ctx)
    assert stage.sync()[0] == vr.VR_OK, vr.vr_last_error(stage.ctx)
    for d in (0, draws - 1) if fits else ():
        part = m.indices[3 * 8 * d:3 * (8 * d + n)]
        rc, ora = vro.process_draw(part, m.vertices, sp, os_, bt, {"max_unique": nu})
        assert cnts[d].cpu().tolist() == [*ora["counters"][:2].tolist(), 0, 0]
        np.testing.assert_array_equal(outs[d].cpu().numpy().view(np.uint32), ora["corners"].view(np.uint32))
    stage.close()
