"""Tiles whose lists are not stored (over the tile cap or the view's list
capacity) scan the survivors of all visible runs: in one item or shared between
several, with few and many runs, fewer and more than a wave's lanes of hits, at
every tile size, lane-owned and not.  Bar: the same bits and work counters as
with lists, and a bounded price."""
import numpy as np
import pytest

import oracle
from scenegen import make_apartment, make_room
from scenegen.walks import random_poses
from tests.geom import pose_at
from tests.gpu_common import gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def _soup(T, seed):
    """Small triangles all over a 16 x 16 pixel frame (64 px focal length) and beyond."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(2.0, 3.0, (T, 1, 1))
    xy = rng.uniform(-0.2, 0.2, (T, 1, 2)) + rng.uniform(-0.03, 0.03, (T, 3, 2))
    pos = np.concatenate([xy * z, np.broadcast_to(-z, (T, 3, 1))], -1).reshape(-1, 3).astype(np.float32)
    return pos, np.arange(3 * T, dtype=np.uint32).reshape(-1, 3), rng.integers(0, 256, (3 * T, 3)).astype(np.uint8)


# runs (256 triangles each) around one, a wave's lanes of counts and beyond; a few views or many
@pytest.mark.parametrize("T", [1, 63, 64, 65, 255, 257, 1000, 16_383, 16_640, 40_000])
@pytest.mark.parametrize("views", [1, 40])
def test_runs_and_parts(ctx, T, views):
    import torch
    pos, idx, col = _soup(T, T)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(40, 24, 40.0, 0.5)
    poses = np.concatenate([pose_at(0.02 * k, 0.01 * (k % 7), 0.01 * k).reshape(1, 12) for k in range(views)])
    note(f"overflow: {T} triangles, {views} views")
    ref = ctx.render(sc, sn, poses, out=ctx.alloc(sn, views, tri=True), tile_size=16, bin_factor=64.0, stats=True)
    want = oracle.render_view(pos, col, idx, 40, 24, poses[0], hfov_deg=40.0, near_m=0.5)
    assert (to_np(ref)["tri"][0] == want["tri"]).all()
    for ts in (8, 16, 32):
        for lane in (False, True):
            for cap in (1, 70):
                o = ctx.alloc(sn, views, tri=True)
                for t in o.values():
                    t.fill_(77)
                ctx.render(sc, sn, poses, out=o, tile_size=ts, tile_cap=cap, bin_factor=64.0, lane_owned_z=lane)
                torch.cuda.synchronize()
                for k in o:
                    assert torch.equal(o[k], ref[k]), (ts, lane, cap, k)
                st = ctx.render(sc, sn, poses, out=o, tile_size=ts, tile_cap=cap, bin_factor=64.0, lane_owned_z=lane,
                                stats=True)["stats"]
                assert st == ref["stats"], (ts, lane, cap)
    assert ctx.get_error() == 0
    ctx.release(sc)


# default capacity: two entries a triangle, so a coarse scene's large frames overflow in part
@pytest.mark.parametrize("n,w,h,near", [(5, 512, 512, 0.01), (1, 1100, 1030, 0.1), (33, 200, 130, 0.01)])
def test_coarse_scene_at_the_default_capacity(ctx, n, w, h, near):
    import torch
    s0 = make_room(seed=81)
    sc = ctx.upload_scene(s0)
    sn = ctx.sensor(w, h, 90.0, near)
    poses = random_poses(s0, n, seed=82)
    note(f"overflow: {n} frames of {w} x {h}")
    outs = []
    for kw in (dict(tile_size=16, bin_factor=64.0), dict(), dict(tile_size=16), dict(tile_size=16, stats=True)):
        o = ctx.alloc(sn, n, tri=True)
        for t in o.values():
            t.fill_(77)
        st = ctx.render(sc, sn, poses, out=o, **kw).pop("stats", None)
        outs.append({k: o[k] for k in ("rgb", "depth", "tri")})
    torch.cuda.synchronize()
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k], outs[0][k]), k
    assert st == ctx.render(sc, sn, poses, out=ctx.alloc(sn, n), tile_size=16, bin_factor=64.0, stats=True)["stats"]
    assert ctx.get_error() == 0
    ctx.release(sc)


@pytest.mark.parametrize("ts", [8, 16])
def test_price_of_a_scan(ctx, ts):
    """Every tile scans its view's survivors: about 20,000 entries where its list has about 200.  With lists this
    launch takes about 0.1 ms; the scan took 0.8 ms at 16 and 1.2 ms at 8 pixels with one block per tile over
    survivors without gaps, and 2.0 and 2.5 ms with one wave over slots with gaps: at most 12 and 16 times the
    lists' time lies between."""
    import torch
    s0 = make_apartment(seed=21, target_T=200_000, jitter_sigma=0.01)
    sc = ctx.upload_scene(s0)
    sn = ctx.sensor(256, 256)
    poses = random_poses(s0, 8, seed=5)
    o = ctx.alloc(sn, 8)
    note(f"overflow: price at {ts} pixels")

    def us(**kw):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = 1e9
        for _ in range(12):
            a.record()
            ctx.render(sc, sn, poses, out=o, tile_size=ts, **kw)
            b.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        return best

    lists, scan = us(), us(tile_cap=64)
    note(f"overflow: {ts} pixels, lists {lists:.0f} us, scan {scan:.0f} us")
    assert scan <= (12 if ts == 16 else 16) * lists
    ctx.release(sc)
