"""Walks of more moves than a workgroup lists: batches whose box, grown by the
longest move and clipped to the grid, is staged whole (up to 4,096 cells) and
ones just larger, at the grid's borders and inside, on grids smaller than the
moves are long, shared by 16, 4 and 1 workgroups, as the per-cell definition
gives them."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev(a):
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int32) if a.dtype == np.uint32 else a).cuda()


# grid, longest move, the cells' box (x0, y0, width, height), agents, batch
CASES = [(200, 19, (80, 90, 26, 26), 600, 300),     # 64 x 64 cells: the largest tile
         (200, 19, (80, 90, 27, 26), 600, 300),     # 65 x 64: from memory
         (200, 19, (0, 0, 45, 45), 600, 300),       # 64 x 64, clipped at two borders
         (200, 19, (170, 155, 30, 45), 600, 300),   # 49 x 64, at the far corner
         (60, 40, (0, 0, 60, 60), 900, 512),        # moves longer than half the grid: the whole field
         (64, 32, (0, 0, 64, 64), 5000, 64),        # 79 batches: four workgroups each
         (65, 32, (0, 0, 65, 65), 900, 512),        # a cell row too many
         (1, 30, (0, 0, 1, 1), 70, 64),             # one cell: no move stays
         (40, 60, (3, 5, 20, 9), 20000, 64)]        # 313 batches: one workgroup each


@pytest.mark.parametrize("num", [1, 19, 20])
def test_few_moves_per_agent(num):
    from paper_1805_08893_amd import vr
    s = W.walk_setup(5, grid=50, agents=700, radius=5, gaussians=3)
    s.moves, s.weights = np.ascontiguousarray(s.moves[:num]), np.ascontiguousarray(s.weights[:num])
    u = W.walk_uniforms(5, 1, 700)
    rc, ref, _ = vro.walk_step(s.keys, s, u, vro.NAIVE)
    assert rc == vro.OK
    stage = vr.GeometryStage(0)
    kin = _dev(s.keys)
    kout = torch.empty_like(kin)
    print(f"case naive, {num} moves", flush=True)
    assert vr.vr_walk_step(stage.ctx, kin, _dev(s.activity), 50, _dev(s.moves), _dev(s.weights), _dev(u), vr.VR_NAIVE, 0,
                           kout) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    np.testing.assert_array_equal(kout.cpu().numpy().view(np.uint32), ref)
    stage.close()


@pytest.mark.parametrize("grid,radius,box,agents,batch", CASES)
@pytest.mark.parametrize("strategy", ["hash", "naive"])
def test_tiles(grid, radius, box, agents, batch, strategy):
    from paper_1805_08893_amd import vr
    s = W.walk_setup(3, grid=grid, agents=agents, radius=radius, gaussians=3)
    assert len(s.weights) > 1024
    rng = np.random.default_rng(grid + radius)
    x, y = rng.integers(box[0], box[0] + box[2], agents), rng.integers(box[1], box[1] + box[3], agents)
    for first in range(0, agents, batch):   # every batch spans the box
        for k, (cx, cy) in enumerate(((box[0], box[1]), (box[0] + box[2] - 1, box[1] + box[3] - 1))):
            if first + k < agents:
                x[first + k], y[first + k] = cx, cy
    keys = (x | y << 16).astype(np.uint32)
    s.activity[rng.random(grid * grid) < 0.3] = 0
    u = W.walk_uniforms(3, 1, agents)
    s.keys = keys
    gs, os_ = (vr.VR_STATIC_HASH, vro.STATIC_HASH) if strategy == "hash" else (vr.VR_NAIVE, vro.NAIVE)
    rc, ref, oc = vro.walk_step(keys, s, u, os_, batch)
    assert rc == vro.OK
    stage = vr.GeometryStage(0)
    kin = _dev(keys)
    kout, cnt = torch.empty_like(kin), torch.zeros(4, dtype=torch.int64, device="cuda")
    print(f"case grid {grid} radius {radius} box {box} agents {agents} {strategy}", flush=True)
    assert vr.vr_walk_step(stage.ctx, kin, _dev(s.activity), grid, _dev(s.moves), _dev(s.weights), _dev(u), gs, batch,
                           kout, cnt) == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    np.testing.assert_array_equal(kout.cpu().numpy().view(np.uint32), ref)
    assert cnt.cpu().tolist()[:2] == oc[:2].tolist()
    stage.close()
