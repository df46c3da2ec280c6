"""Work items of the 16-pixel tiles' raster in launches below and above the number
of tiles from which items hold twice the entries: lists around one, two and three
items, against 8-pixel tiles and the oracle.  Bar: the same bits."""
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


@pytest.mark.parametrize("views", [2, 2100])      # 16 tiles each: 32, and 33600 in one launch
@pytest.mark.parametrize("n", [127, 128, 129, 256, 257, 384, 385, 700])
def test_items(ctx, views, n):
    import torch
    note(f"segments: {views} views, {n} triangles on a tile")
    rng = np.random.default_rng(n)
    z = rng.uniform(2.0, 3.0, (n, 3))
    p = 24.0 + rng.uniform(-3, 3, (n, 1, 2)) + rng.uniform(-3, 3, (n, 3, 2))     # pixels 18 to 30: one tile
    xy = (p - 32.0) / 32.0 * z[..., None]
    pos = np.concatenate([xy * [1.0, -1.0], -z[..., None]], -1).reshape(-1, 3).astype(np.float32)
    idx = np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)
    col = rng.integers(0, 256, (len(pos), 3)).astype(np.uint8)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(64, 64, 90.0, 1.0)
    poses = np.repeat(pose_at(0, 0, 0).reshape(1, 12), views, 0)
    ref = ctx.render(sc, sn, poses[:1], out=ctx.alloc(sn, 1, tri=True), tile_size=8)
    want = oracle.render_view(pos, col, idx, 64, 64, poses[0], near_m=1.0)
    assert (to_np(ref)["tri"][0] == want["tri"]).all()
    o = ctx.alloc(sn, views, tri=True)
    for t in o.values():
        t.fill_(77)
    ctx.render(sc, sn, poses, out=o, tile_size=16, one_sequence=True)
    for k in o:
        assert bool((o[k] == ref[k]).all()), k
    assert ctx.get_error() == 0
    ctx.release(sc)
