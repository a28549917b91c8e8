"""Walk steps of agents spread over the largest grid: boxes of up to 32,768
cells with moves so long that a window would hold two cells a side, as the
per-cell definition gives them."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRID = 32768


@pytest.mark.parametrize("radius,agents,batch", [(31, 40, 512), (31, 700, 2), (16, 300, 300)])
def test_agents_over_the_whole_grid(radius, agents, batch):
    from paper_1805_08893_amd import vr
    rng = np.random.default_rng(radius)
    d = rng.integers(-radius, radius + 1, (120, 2))
    moves = np.unique(np.concatenate([d, [[radius, 0], [0, -radius], [-radius, radius]]]), axis=0)
    moves = np.ascontiguousarray(moves[(moves != 0).any(axis=1)], dtype=np.int8)
    weights = rng.random(len(moves), dtype=np.float32)
    x, y = rng.integers(0, GRID, agents).astype(np.uint32), rng.integers(0, GRID, agents).astype(np.uint32)
    x[:4], y[:4] = (0, GRID - 1, 0, GRID - 1), (0, 0, GRID - 1, GRID - 1)
    keys = x | y << np.uint32(16)
    act = np.zeros(GRID * GRID, np.float32)   # activity around the agents only: most pages stay untouched
    dev = torch.zeros(GRID * GRID, dtype=torch.float32, device="cuda")
    r = np.arange(-radius, radius + 1)
    tx, ty = x.astype(np.int64)[:, None, None] + r, y.astype(np.int64)[:, None, None] + r[:, None]
    tx, ty = np.broadcast_arrays(tx, ty)
    at = (ty * GRID + tx)[(tx >= 0) & (ty >= 0) & (tx < GRID) & (ty < GRID)]
    at = np.unique(at)
    val = rng.random(len(at), dtype=np.float32)
    act[at] = val
    dev[torch.from_numpy(at).cuda()] = torch.from_numpy(val).cuda()
    u = W.walk_uniforms(5, 1, agents)
    setup = W.WalkSetup(GRID, act, moves, weights, keys, 5)
    rc, ref, oc = vro.walk_step(keys, setup, u, vro.STATIC_HASH, batch)
    assert rc == vro.OK
    stage = vr.GeometryStage(0)
    kin = torch.from_numpy(keys.view(np.int32)).cuda()
    kout = torch.empty_like(kin)
    cnt = torch.zeros(4, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    print(f"case radius {radius} agents {agents} batch {batch}", flush=True)
    assert vr.vr_walk_step(stage.ctx, kin, dev, GRID, torch.from_numpy(moves).cuda(), torch.from_numpy(weights).cuda(),
                           torch.from_numpy(u).cuda(), vr.VR_STATIC_HASH, batch, kout, cnt) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    np.testing.assert_array_equal(kout.cpu().numpy().view(np.uint32), ref)
    assert cnt.cpu().tolist()[:2] == oc[:2].tolist()
    stage.close()
