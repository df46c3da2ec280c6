"""Views of more tiles than are binned at once (windows of whole tile rows), alone
and in a batch with small ones: square, wide and tall, small triangles and ones
that cover many windows.  Bar: the same bits as without lists (every tile over its
cap) and as the oracle, and a price that follows the pixels."""
import numpy as np
import pytest

import oracle
from scenegen import make_apartment, make_room
from scenegen.walks import random_poses
from tests.gpu_common import gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


# tiles: 2048 (the limit) and 2112 of 16 pixels; 8 pixels: 512 a row, rows of 1, 2
@pytest.mark.parametrize("w,h,ts", [(512, 1024, 16), (528, 1024, 16), (1024, 1040, 16), (4096, 200, 8), (9, 4096, 8),
                                    (16, 4096, 8), (40, 4096, 8), (700, 650, 8), (2100, 40, 8), (1600, 1500, 32)])
@pytest.mark.parametrize("tri", [2_000, 40_000])
def test_windows(ctx, w, h, ts, tri):
    import torch
    s0 = make_room(seed=91) if tri == 2_000 else make_apartment(seed=92, target_T=tri, jitter_sigma=0.01)
    sc = ctx.upload_scene(s0)
    sn = ctx.sensor(w, h, 90.0, 0.2)
    small = ctx.sensor(48, 40)
    poses = random_poses(s0, 3, seed=93)
    note(f"large views: {w} x {h}, {ts}-pixel tiles, {tri} triangles")

    def batch(**kw):
        outs = [ctx.alloc(s, 1, tri=True) for s in (sn, small, sn)]
        for o in outs:
            for t in o.values():
                t.fill_(77)
        ctx.render_batch([(sc, s, poses[k], o["rgb"], o["depth"], o["tri"]) for k, (s, o) in
                          enumerate(zip((sn, small, sn), outs))], tile_size=ts, **kw)
        torch.cuda.synchronize()
        return outs

    ref, got, default = batch(tile_cap=1), batch(bin_factor=64.0), batch()
    for a, b, c in zip(ref, got, default):
        for k in a:
            assert torch.equal(a[k], b[k]) and torch.equal(a[k], c[k]), k
    if w * h <= 600_000:
        o = oracle.render_view(s0.positions, s0.colors, s0.indices, w, h, poses[0], near_m=0.2)
        assert (to_np(got[0])["tri"][0] == o["tri"]).all()
    assert ctx.get_error() == 0
    ctx.release(sc)


def test_price_follows_the_pixels(ctx):
    """A 2048 x 2048 frame of a 2k-triangle room against a 512 x 512 one, which has a sixteenth of its tiles: the
    windows take 8 times as long; a global atomic per tile and survivor took 42 times as long."""
    import torch
    s0 = make_room(seed=11)
    sc = ctx.upload_scene(s0)
    p = random_poses(s0, 1, seed=5)

    def us(size, near):
        sn = ctx.sensor(size, size, 90.0, near)
        o = ctx.alloc(sn, 1)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = 1e9
        for _ in range(12):
            a.record()
            ctx.render(sc, sn, p, out=o, tile_size=16)
            b.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        return best

    few, many = us(512, 0.1), us(2048, 0.1)
    note(f"large views: 512 x 512 {few:.0f} us, 2048 x 2048 {many:.0f} us")
    assert many <= 20 * few
    ctx.release(sc)
