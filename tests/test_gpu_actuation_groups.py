"""Actuation and free-space queries at the sizes where their launches change
(lanes per agent or point) and in obstacle sets that overflow a group's list
of candidate segments or span more grid rows than a group has lanes.  Bar: as
in test_gpu_actuation.py, bit-identical to the oracle."""
import math

import numpy as np
import pytest

import oracle
from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu
C10, S10 = math.cos(math.radians(10.0)), math.sin(math.radians(10.0))


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def _obstacles(n, extent, length, seed):
    rng = np.random.default_rng(seed)
    a = rng.uniform(0.0, extent, (n, 2))
    t = rng.uniform(0.0, 2 * math.pi, n)
    d = length * rng.uniform(0.2, 1.0, n)
    d[::17] = 0.0                                    # point obstacles
    return np.concatenate([a, a + np.stack([np.cos(t) * d, np.sin(t) * d], 1)], 1).astype(np.float32)


# (agents, forward m, segments, extent m, segment length m)
@pytest.mark.parametrize("n,step,nseg,extent,length", [
    (1, 0.25, 400, 6.0, 0.5), (5, 0.25, 400, 6.0, 0.5), (8192, 0.25, 150, 9.0, 0.5), (8193, 0.25, 150, 9.0, 0.5),
    (32768, 0.25, 60, 9.0, 0.5), (32769, 0.25, 60, 9.0, 0.5),
    (300, 0.25, 3000, 2.0, 0.3),      # hundreds of candidates within one step: lists overflow
    (300, 40.0, 300, 60.0, 0.05),     # a step across more grid rows than a group has lanes
    (9000, 12.0, 200, 30.0, 0.05)])
def test_group_sizes(ctx, n, step, nseg, extent, length):
    import torch
    note(f"actuation groups: {n} agents, {step} m, {nseg} segments")
    seg = _obstacles(nseg, extent, length, 5)
    nav, none = ctx.nav_upload(seg), ctx.nav_upload(np.zeros((0, 4), np.float32))
    rng = np.random.default_rng(n + nseg)
    yaw = rng.uniform(0.0, 2 * math.pi, n)
    ag = np.concatenate([rng.uniform(-0.3, extent + 0.3, (n, 2)), np.stack([-np.sin(yaw), -np.cos(yaw)], 1)], 1)
    act = rng.choice([0, 1, 1, 1, 2, 3, 9], n).astype(np.uint8)
    act[0] = 1
    free = rng.random(n) < 0.1                       # agents of a scene without obstacles
    free[0] = False
    t = torch.from_numpy(ag.copy()).cuda()
    hit = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    poses = torch.empty((n, 12), dtype=torch.float32, device="cuda")
    ctx.actuate([none if f else nav for f in free], t, torch.from_numpy(act).cuda(), hit, poses, 1.5,
                ctx.actuation(0.1, step, 10.0))
    got, ghit, gposes = t.cpu().numpy(), hit.cpu().numpy(), poses.cpu().numpy()
    pick = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n),
                                     rng.integers(0, n, min(n, 3000))]))
    oact = np.where(act > 3, 0, act)
    for sel, s in ((pick[~free[pick]], seg), (pick[free[pick]], np.zeros((0, 4), np.float32))):
        if sel.size:
            want, whit = oracle.actuate(s, ag[sel], oact[sel], 0.1, step, C10, S10)
            assert np.array_equal(got[sel].view(np.uint64), want.view(np.uint64))
            assert np.array_equal(ghit[sel], whit.astype(np.uint8))
            assert np.array_equal(gposes[sel], oracle.agent_pose(want, 1.5))
    assert set(np.unique(ghit)) <= {0, 1}
    ctx.nav_release(nav)
    ctx.nav_release(none)


@pytest.mark.parametrize("n,radius,nseg", [(1, 0.1, 200), (63, 0.1, 200), (131072, 0.1, 200), (131073, 0.1, 200),
                                           (5000, 4.0, 500), (5000, 0.01, 4000)])
def test_free_space_sizes(ctx, n, radius, nseg):
    import torch
    note(f"free space: {n} points, radius {radius}, {nseg} segments")
    seg = _obstacles(nseg, 20.0, 0.4, 9)
    nav = ctx.nav_upload(seg)
    rng = np.random.default_rng(n)
    pts = rng.uniform(-5.0, 25.0, (n, 2))
    got = ctx.nav_free(nav, torch.from_numpy(pts).cuda(), radius).cpu().numpy().astype(bool)
    pick = np.unique(np.concatenate([np.arange(min(n, 100)), np.arange(max(0, n - 100), n),
                                     rng.integers(0, n, min(n, 5000))]))
    assert np.array_equal(got[pick], oracle.nav_free(seg, pts[pick], radius))
    ctx.nav_release(nav)
