"""Dynamic batches with a triangle cap far above what the unique budget lets a
closed mesh's batch hold: units of few distinct indices fill the cap and are
deduplicated in several chunks, ordinary ones in one; every output against the
oracle."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# a sort's unit holds at most 8,192 indices
@pytest.mark.parametrize("name,bt,nu", [(n, b, u) for n in ("dyn_hash", "dyn_phash", "dyn_sort")
                                        for b, u in ((256, 64), (1024, 64), (1024, 256), (4096, 256))
                                        if n != "dyn_sort" or b < 4096])
@pytest.mark.parametrize("kind", ["grid", "few"])
def test_outputs(name, bt, nu, kind):
    from paper_1805_08893_amd import vr
    m = W.grid_mesh(61, 75, 4, "hilbert")
    ind = m.indices.copy()
    if kind == "few":   # runs of triangles over nu - 1 vertices each, longer than the cap
        t = np.arange(m.num_tris, dtype=np.uint32)
        ind = (t[:, None] // (2 * bt + 7) * nu + (t[:, None] * 7 + np.arange(3, dtype=np.uint32) * 5) % (nu - 1)).astype(np.uint32)
        ind = np.ascontiguousarray(ind.reshape(-1))
        assert ind.max() < m.num_verts
    sp = W.shader_for_mesh(m, W.SHADER_MVP, 4)
    rc, ora = vro.process_draw(ind, m.vertices, sp, vro.STRATEGY_NAMES.index(name), bt, {"max_unique": nu})
    assert rc == vro.OK
    inv, units = (int(x) for x in ora["counters"][:2])
    idx, vtx = torch.from_numpy(ind.view(np.int32)).cuda(), torch.from_numpy(m.vertices).cuda()
    stage = vr.GeometryStage(0)
    gs = vr.STRATEGIES[name]
    print(f"case {name} {bt}/{nu} {kind}", flush=True)
    for want in (dict(corners=True), dict(corners=False, tris=True, verts=True),
                 dict(corners=True, tris=True, verts=True, local_idx=True, units=True)):
        res = stage.draw(idx, vtx, sp, gs, bt, dict(max_unique=nu), **want)
        assert stage.sync()[0] == vr.VR_OK
        assert res["counters"].cpu().tolist() == [inv, units, 0, 0]
        for key in ("corners", "tris", "local_idx"):
            if want.get(key):
                a, b = res[key].cpu().numpy(), ora[key]
                np.testing.assert_array_equal(a.view(b.dtype if key != "corners" else np.uint32), b if key != "corners" else b.view(np.uint32))
        if want.get("verts"):
            np.testing.assert_array_equal(res["verts"].cpu().numpy()[:inv].view(np.uint32), ora["verts"].view(np.uint32))
        if want.get("units"):
            np.testing.assert_array_equal(res["unit_offsets"].cpu().numpy().view(np.uint32)[:units + 1], ora["unit_offsets"])
    stage.close()
