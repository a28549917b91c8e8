"""Deduplication from registers: units whose corner count sits at, just below
and just above the corners a workgroup holds at once (4 per thread), units of
several such chunks up to the most a thread may own, and the sort of one to
eight rounds of distinct indices; with corners only (ids in any order) and
with every output (canonical ids), bitwise against the oracle."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

S = vro
CASES = [  # strategy, batch_tris, max_unique, wg_size
    (S.STATIC_HASH, 85, 0, 64), (S.STATIC_HASH, 86, 0, 64), (S.DYN_HASH, 85, 64, 0), (S.DYN_HASH, 86, 64, 64),
    (S.DYN_HASH, 171, 512, 128), (S.DYN_HASH, 341, 256, 64), (S.DYN_HASH, 682, 512, 64), (S.DYN_HASH, 682, 512, 0),
    (S.DYN_HASH, 1024, 700, 1024), (S.DYN_PHASH, 342, 256, 256), (S.DYN_PHASH, 341, 256, 64),
    (S.DYN_SORT, 341, 256, 0), (S.DYN_SORT, 341, 512, 256), (S.DYN_SORT, 170, 510, 64), (S.DYN_SORT, 170, 200, 128),
    (S.DYN_SORT, 682, 2046, 256), (S.STATIC_SORT, 256, 0, 0), (S.STATIC_SORT, 256, 0, 1024), (S.DYN_SORT, 1, 3, 0),
]


def _meshes():
    rng = np.random.default_rng(23)
    V = 3000
    return (W.take_prefix(W.icosphere_mesh(5, 6, "hilbert", swap_frac=0.05), 6001),
            W.Mesh("spread", rng.integers(0, V, 3 * 2049).astype(np.uint32), W.grid_mesh(60, 50, 9).vertices))


@pytest.mark.parametrize("strategy,bt,nu,wg", CASES)
def test_units_at_register_chunk_edges(strategy, bt, nu, wg):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    for mesh in _meshes():
        print(f"case strategy={strategy} bt={bt} nu={nu} wg={wg} mesh={mesh.name} T={mesh.num_tris}", flush=True)
        sp = W.shader_for_mesh(mesh, W.SHADER_PHONG, 3, num_lights=2)
        rc, ora = vro.process_draw(mesh.indices, mesh.vertices, sp, strategy, bt, {"max_unique": nu})
        assert rc == 0
        idx = torch.from_numpy(mesh.indices.view(np.int32)).cuda()
        vtx = torch.from_numpy(mesh.vertices).cuda()
        inv, units = int(ora["counters"][0]), int(ora["counters"][1])
        for every in (False, True):
            res = stage.draw(idx, vtx, sp, strategy, bt, dict(max_unique=nu, wg_size=wg), corners=True, tris=every,
                             verts=every, local_idx=every, units=every)
            st, total = stage.sync()
            assert st == vr.VR_OK and total == inv
            got = {k: v.cpu().numpy() for k, v in res.items()}
            assert got["counters"][:2].tolist() == [inv, units]
            np.testing.assert_array_equal(got["corners"].view(np.uint32), ora["corners"].view(np.uint32))
            if every:
                np.testing.assert_array_equal(got["local_idx"].view(np.uint16), ora["local_idx"])
                np.testing.assert_array_equal(got["tris"].view(np.uint32), ora["tris"])
                np.testing.assert_array_equal(got["verts"][:inv].view(np.uint32), ora["verts"].view(np.uint32))
                np.testing.assert_array_equal(got["unit_invocations"][:units].view(np.uint32), ora["unit_invocations"])
    stage.close()
