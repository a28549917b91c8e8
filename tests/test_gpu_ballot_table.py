"""The rounds' table: batches of one index, of 64 and 65 distinct indices, of
all distinct ones, of indices that collide in the round's 256 slots, with a
round ending inside, at and after a group of 21 triangles, against the oracle
bit for bit (static and dynamic, corners only and every output)."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _colliding(n, V):
    """n indices below V whose hash falls into the same 1/256 of the range."""
    k = np.arange(V, dtype=np.uint64)
    return k[((k * 0x9E3779B1 & 0xFFFFFFFF) >> 24) == 7][:n].astype(np.uint32)


def _streams(V):
    rng = np.random.default_rng(41)
    few = _colliding(200, V)
    yield "one", np.full(3 * 400, 9, np.uint32)
    for d in (3, 63, 64, 65, 66, 127):
        yield f"cycle{d}", (np.arange(3 * 400) % d).astype(np.uint32)
    yield "distinct", np.arange(3 * 400, dtype=np.uint32)
    yield "colliding", few[rng.integers(0, len(few), 3 * 400)]
    yield "distinct_colliding", np.resize(few, 3 * 200)
    yield "mixed", np.where(rng.random(1200) < 0.5, rng.integers(0, V, 1200), few[rng.integers(0, 70, 1200)]).astype(np.uint32)


@pytest.mark.parametrize("strategy,bt,nu", [(vro.STATIC_BALLOT, 1, 0), (vro.STATIC_BALLOT, 21, 0),
                                            (vro.STATIC_BALLOT, 22, 0), (vro.STATIC_BALLOT, 64, 0),
                                            (vro.STATIC_BALLOT, 1024, 0), (vro.DYN_BALLOT, 85, 64),
                                            (vro.DYN_BALLOT, 512, 200)])
def test_rounds(strategy, bt, nu):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    base = W.grid_mesh(260, 250, 3)
    sp = W.shader_for_mesh(base, W.SHADER_MVP, 3)
    vtx = torch.from_numpy(base.vertices).cuda()
    for name, ind in _streams(base.num_verts):
        print(f"case {strategy} {bt}/{nu} {name}", flush=True)
        rc, ora = vro.process_draw(ind, base.vertices, sp, strategy, bt, {"max_unique": nu})
        assert rc == 0
        inv, units = int(ora["counters"][0]), int(ora["counters"][1])
        idx = torch.from_numpy(ind.view(np.int32).copy()).cuda()
        for every in (False, True):
            res = stage.draw(idx, vtx, sp, strategy, bt, dict(max_unique=nu), corners=True, tris=every, verts=every,
                             local_idx=every, units=every)
            st, total = stage.sync()
            assert st == vr.VR_OK and total == inv
            got = {k: v.cpu().numpy() for k, v in res.items()}
            assert got["counters"][:2].tolist() == [inv, units]
            np.testing.assert_array_equal(got["corners"].view(np.uint32), ora["corners"].view(np.uint32))
            if every:
                np.testing.assert_array_equal(got["local_idx"].view(np.uint16), ora["local_idx"])
                np.testing.assert_array_equal(got["tris"].view(np.uint32), ora["tris"])
                np.testing.assert_array_equal(got["unit_offsets"][:units + 1].view(np.uint32), ora["unit_offsets"])
    stage.close()
