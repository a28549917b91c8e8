"""The planner's short windows and lists: budgets where the cut lies before,
at and after a third of the budget, windows more and less than twice over it
within one block of starts, budgets above the primitive cap, one hub index in
every triangle, and streams whose length is a block of starts, one less and
one more; plans equal the sequential greedy chain."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _streams():
    rng = np.random.default_rng(31)
    spread = rng.integers(0, 60000, 3 * 2600).astype(np.uint32)
    near = (np.repeat(np.arange(2600), 3) // 9 + rng.integers(0, 12, 3 * 2600)).astype(np.uint32)
    mixed = np.where(np.repeat(np.arange(2600) // 150 % 2, 3) == 0, spread, near).astype(np.uint32)
    hub = spread.copy()
    hub[::3] = 5
    return {"spread": spread, "near": near, "mixed": mixed, "hub": hub}


@pytest.mark.parametrize("nu,tmax", [(3, 2), (4, 7), (100, 256), (256, 341), (85, 512), (700, 256), (300, 900)])
@pytest.mark.parametrize("T", [511, 512, 513, 1023, 1024, 1025, 2600])
def test_plans(nu, tmax, T):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    for name, idx in _streams().items():
        print(f"case plan {nu}/{tmax} {name} T={T}", flush=True)
        exp = vro.plan_dynamic(idx[:3 * T], 60000, nu, tmax)
        dev = torch.from_numpy(idx[:3 * T].view(np.int32).copy()).cuda()
        plan = torch.empty(T + 2, dtype=torch.int32, device="cuda")
        assert vr.vr_plan_dynamic(stage.ctx, dev, 60000, nu, tmax, plan) == vr.VR_OK
        assert stage.sync()[0] == vr.VR_OK
        got = plan.cpu().numpy().view(np.uint32)
        assert int(got[0]) == len(exp) - 1
        np.testing.assert_array_equal(got[1:len(exp) + 1], exp)
    stage.close()
