"""The walk's move lists and windows: move counts at the edges of the listed
search (one move, fewer than the options kept, the most listed, one more),
signed, zero, tied and infinite weights and activities with NaN among them,
boxes of one window and of many, batches shared by 16, 4 and 1 workgroups, and
keys updated in place, exactly as the per-cell definition gives them."""
import numpy as np
import pytest

from oracle import vro
from paper_1805_08893_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev(a):
    a = np.ascontiguousarray(a)
    return torch.from_numpy(a.view(np.int32) if a.dtype == np.uint32 else a).cuda()


def _cells(setup, strategy, batch):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    kin = _dev(setup.keys)
    kout = torch.empty_like(kin)
    st = vr.vr_walk_step(stage.ctx, kin, _dev(setup.activity), setup.grid, _dev(setup.moves), _dev(setup.weights),
                         _dev(W.walk_uniforms(setup.seed, 1, len(setup.keys))), strategy, batch, kout)
    assert st == vr.VR_OK and stage.sync()[0] == vr.VR_OK
    stage.close()
    return kout.cpu().numpy()


def _run(setup, strategy, batch, in_place=False):
    from paper_1805_08893_amd import vr
    stage = vr.GeometryStage(0)
    u = W.walk_uniforms(setup.seed, 1, len(setup.keys))
    kin = _dev(setup.keys)
    kout = kin if in_place else torch.empty_like(kin)
    cnt = torch.zeros(4, dtype=torch.int64, device="cuda")
    st = vr.vr_walk_step(stage.ctx, kin, _dev(setup.activity), setup.grid, _dev(setup.moves), _dev(setup.weights),
                         _dev(u), vr.VR_NAIVE if strategy == "naive" else vr.VR_STATIC_HASH, batch, kout, cnt)
    assert st == vr.VR_OK
    assert stage.sync()[0] == vr.VR_OK
    rc, ref, oc = vro.walk_step(setup.keys, setup, u, vro.NAIVE if strategy == "naive" else vro.STATIC_HASH, batch)
    assert rc == vro.OK
    np.testing.assert_array_equal(kout.cpu().numpy().view(np.uint32), ref)
    assert cnt.cpu().tolist()[:2] == oc[:2].tolist()
    stage.close()


@pytest.mark.parametrize("strategy,batch", [("naive", 0), ("hash", 512), ("hash", 37)])
@pytest.mark.parametrize("num", [1, 7, 8, 17, 1023, 1024, 1025])
def test_move_counts(strategy, batch, num):
    s = W.walk_setup(5, grid=70, agents=1500, radius=19, gaussians=3)
    keep = np.linspace(0, len(s.weights) - 1, num).astype(int)
    s.moves, s.weights = np.ascontiguousarray(s.moves[keep]), np.ascontiguousarray(s.weights[keep])
    print(f"case {strategy} {batch} moves {num}", flush=True)
    _run(s, strategy, batch)


@pytest.mark.parametrize("kind", ["tied", "signed", "zero", "inf", "nan"])
@pytest.mark.parametrize("strategy,batch", [("naive", 0), ("hash", 300)])
def test_values(kind, strategy, batch):
    s = W.walk_setup(6, grid=60, agents=2500, radius=7, gaussians=3)
    rng = np.random.default_rng(4)
    if kind == "tied":
        s.activity[:] = np.float32(0.25)
        s.weights = rng.choice(np.float32([0.5, 0.25]), len(s.weights))
    elif kind == "signed":   # products above -1 are kept, below they are not
        s.activity *= rng.choice(np.float32([-1, 1]), len(s.activity))
        s.weights *= rng.choice(np.float32([-3, 1]), len(s.weights))
    elif kind == "zero":
        s.activity[rng.random(len(s.activity)) < 0.9] = 0
        s.weights[::3] = 0
        s.weights[1::3] = -0.0
    elif kind == "inf":
        s.activity[::501] = np.inf
    else:
        s.activity[::7] = np.nan
        s.weights[::5] = np.nan
        from paper_1805_08893_amd import vr
        np.testing.assert_array_equal(_cells(s, vr.VR_STATIC_HASH, batch or 64), _cells(s, vr.VR_NAIVE, 0))
        return
    print(f"case {kind} {strategy} {batch}", flush=True)
    _run(s, strategy, batch)


@pytest.mark.parametrize("agents,grid,order,batch,in_place", [
    (300, 256, "random", 512, False), (3000, 250, "random", 300, False), (3000, 250, "hilbert", 300, True),
    (9000, 256, "random", 64, False), (9000, 300, "hilbert", 32, False), (2000, 40, "hilbert", 512, False)])
def test_boxes_and_workgroups_per_batch(agents, grid, order, batch, in_place):
    s = W.walk_setup(8, grid=grid, agents=agents, radius=12, gaussians=4, order=order)
    print(f"case agents {agents} grid {grid} {order} batch {batch} in place {in_place}", flush=True)
    _run(s, "hash", batch, in_place)
