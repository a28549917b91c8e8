"""The piece each workgroup takes (contiguous runs per XCD) covers every unit
exactly once: draws around 1 to 17 pieces (multiples of the XCD count and next
to them), a triangle more and less, and dynamic draws with
more batches than the fewest, against the oracle bit for bit."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [(vro.NAIVE, 1, 0), (vro.STATIC_HASH, 5, 0), (vro.STATIC_BALLOT, 4, 0), (vro.MULTI, 1, 0),
         (vro.DYN_HASH, 8, 9), (vro.DYN_BALLOT, 8, 9)]


@pytest.mark.parametrize("strategy,bt,nu", CASES)
def test_pieces_cover_every_unit(strategy, bt, nu):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    whole = W.grid_mesh(31, 29, 4, "hilbert")
    sp = W.shader_for_mesh(whole, W.SHADER_PHONG, 4, num_lights=1)
    per = {vro.NAIVE: 86, vro.MULTI: 86}.get(strategy, bt)
    sizes = sorted({max(1, min(whole.num_tris, per * k + d)) for k in (1, 2, 7, 8, 9, 15, 16, 17) for d in (-1, 0, 1)})
    for T in sizes:
        mesh = W.take_prefix(whole, T)
        print(f"case strategy={strategy} T={T}", flush=True)
        rc, ora = vro.process_draw(mesh.indices, mesh.vertices, sp, strategy, bt, {"max_unique": nu}, local_idx=False)
        assert rc == 0
        idx = torch.from_numpy(mesh.indices.view(np.int32)).cuda()
        vtx = torch.from_numpy(mesh.vertices).cuda()
        res = stage.draw(idx, vtx, sp, strategy, bt, dict(max_unique=nu))
        st, total = stage.sync()
        assert st == vr.VR_OK and total == int(ora["counters"][0])
        np.testing.assert_array_equal(res["corners"].cpu().numpy().view(np.uint32), ora["corners"].view(np.uint32))
        assert res["counters"].cpu().tolist()[:2] == [int(x) for x in ora["counters"][:2]]
    stage.close()
