"""Small triangles that cover no pixel centre are dropped by the setup unless the
view's work is counted: the frames of a launch that drops them against one that
does not and against the oracle.  Bar: the same bits.  Vertices lie on quarters
of a pixel, so edges and corners meet pixel centres (the fill rule decides) in
both orientations, with boxes of one to a few centres, some cut by the view's
border, and extents on both sides of 8 px."""
import numpy as np
import pytest

import oracle
from tests.geom import pose_at
from tests.gpu_common import gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


@pytest.mark.parametrize("w,h", [(0.5, 0.5), (1, 1), (2, 1), (1, 2), (2, 2), (4, 1), (1, 4), (5, 1), (3, 2), (8, 0.5),
                                 (0.5, 8), (8.25, 1), (1, 8.25), (30, 1)])
@pytest.mark.parametrize("border", [False, True])
def test_frames_do_not_change(ctx, w, h, border):
    import torch
    note(f"small triangles: {w} x {h} px, border {border}")
    rng = np.random.default_rng([int(4 * w), int(4 * h), border])
    n, size = 1500, 64
    at = rng.integers(-8, 4 * size + 8, (n, 1, 2)) / 4.0
    if border:   # within two pixels of an edge of the view
        side = rng.integers(0, 2, n)
        at[np.arange(n), 0, side] = rng.integers(0, 2, n) * size + rng.integers(-8, 9, n) / 4.0
    px = at + np.rint(rng.uniform(-0.5, 0.5, (n, 3, 2)) * [4 * w, 4 * h]) / 4.0
    xy = (px - size / 2) / (size / 2) * 2.0           # 90 degrees, depth 2: exact in fp32
    pos = np.concatenate([xy * [1.0, -1.0], np.full((n, 3, 1), -2.0)], -1).reshape(-1, 3).astype(np.float32)
    idx = np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)
    col = rng.integers(0, 256, (len(pos), 3)).astype(np.uint8)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(size, size, 90.0, 1.0)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    want = oracle.render_view(pos, col, idx, size, size, pose[0], near_m=1.0)
    counted = ctx.render(sc, sn, pose, out=ctx.alloc(sn, 1, tri=True), tile_size=16, stats=True)
    for ts in (8, 16, 32, 0):
        o = ctx.alloc(sn, 1, tri=True)
        ctx.render(sc, sn, pose, out=o, tile_size=ts)
        for k in o:
            assert torch.equal(o[k], counted[k]), (ts, k)
        assert (to_np(o)["tri"][0] == want["tri"]).all(), ts
    assert ctx.get_error() == 0
    ctx.release(sc)
