"""Planning where places in the hash table collide: grids whose rows nearly
coincide under the hash, in windows of every cap class, and random windows that
fill the table, against the sequential chain."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,order", [(341, 80, "hilbert"), (377, 70, "hilbert"), (233, 100, "hilbert"),
                                         (1341, 30, "hilbert"), (1341, 30, "random")])
@pytest.mark.parametrize("nu,tmax", [(64, 128), (100, 256), (256, 512), (300, 1024), (1024, 2048), (2048, 4096)])
def test_plan(nx, ny, order, nu, tmax):
    from paper_1805_08893_amd import vr
    m = W.grid_mesh(nx, ny, 4, order)
    ref = vro.plan_dynamic(m.indices, m.num_verts, nu, tmax)
    stage = vr.GeometryStage(0)
    idx = torch.from_numpy(m.indices.view(np.int32)).cuda()
    plan = torch.zeros(m.num_tris + 2, dtype=torch.int32, device="cuda")
    print(f"case {nx} x {ny} {order} {tmax}/{nu}", flush=True)
    assert vr.vr_plan_dynamic(stage.ctx, idx, m.num_verts, nu, tmax, plan) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    got = plan.cpu().numpy()
    assert got[0] == len(ref) - 1
    np.testing.assert_array_equal(got[1:1 + len(ref)].view(np.uint32), ref)
    stage.close()
