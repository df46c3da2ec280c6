"""Triangles whose edges do not fit the packed 16-bit form, in 32-bit and in 64-bit
edge values, around the sizes where one gives way to the other, at 16-pixel tiles.
Bar: the same bits and work counters as 8-pixel tiles, the triangles of the oracle."""
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


@pytest.mark.parametrize("size", [120, 140, 500, 900, 1050, 1100, 1200, 2000, 3000, 20_000, 400_000])
@pytest.mark.parametrize("tri", [1, 90])
def test_sizes(ctx, size, tri):
    import torch
    note(f"unpacked: {tri} triangles of {size} px")
    rng = np.random.default_rng(size + tri)
    z = rng.uniform(2.0, 3.0, (tri, 1, 1))
    p = 32.0 + rng.uniform(-60, 60, (tri, 1, 2)) + rng.uniform(-0.5, 0.5, (tri, 3, 2)) * size
    xy = (p - 32.0) / 32.0 * z
    pos = np.concatenate([xy * [1.0, -1.0], np.broadcast_to(-z, (tri, 3, 1))], -1).reshape(-1, 3).astype(np.float32)
    idx = np.arange(3 * tri, dtype=np.uint32).reshape(-1, 3)
    col = rng.integers(0, 256, (3 * tri, 3)).astype(np.uint8)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(75, 61, 90.0, 1.0)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    outs = [ctx.render(sc, sn, pose, out=ctx.alloc(sn, 1, tri=True), tile_size=ts, stats=True) for ts in (16, 8)]
    plain = ctx.render(sc, sn, pose, out=ctx.alloc(sn, 1, tri=True), tile_size=16)
    torch.cuda.synchronize()
    for k in ("rgb", "depth", "tri"):
        assert torch.equal(outs[0][k], outs[1][k]) and torch.equal(outs[0][k], plain[k]), k
    assert outs[0]["stats"] == outs[1]["stats"]
    want = oracle.render_view(pos, col, idx, 75, 61, pose[0], near_m=1.0)
    assert (to_np(plain)["tri"][0] == want["tri"]).all()
    assert ctx.get_error() == 0
    ctx.release(sc)
