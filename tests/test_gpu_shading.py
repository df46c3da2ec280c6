"""Shading of the visible triangles: the weights of a pixel from near and far
vertices (24-bit and 64-bit edge functions), both orientations and near-clipped
triangles, coloured and textured, against the oracle; and the blocks that shade
one, two or four bands of a view, whose frames must be the same bits.  Bar for
colour: within 1 of 255, as everywhere; depth 1e-5, ids exact."""
import numpy as np
import pytest

import oracle
from scenegen import configs, with_texture
from tests.geom import pose_at
from tests.gpu_common import gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


@pytest.mark.parametrize("size", [3, 40, 127, 129, 400, 9000])   # px: 64 px from the pixel is the form's border
@pytest.mark.parametrize("textured", [False, True])
@pytest.mark.parametrize("clipped", [False, True])
def test_weights_against_the_oracle(ctx, size, textured, clipped):
    note(f"shading: {size} px, textured {textured}, clipped {clipped}")
    rng = np.random.default_rng([size, textured, clipped])
    n = 300
    z = rng.uniform(2.0, 3.0, (n, 3))
    if clipped:
        z[:, 2] = rng.uniform(-1.0, 0.9, n)      # one vertex behind the near plane at 1 m
    c = 24.0 + rng.uniform(-20, 20, (n, 2))
    p = c[:, None] + rng.uniform(-0.5, 0.5, (n, 3, 2)) * size
    xy = (p - 32.0) / 32.0 * np.maximum(z, 1.0)[..., None]
    pos = np.concatenate([xy * [1.0, -1.0], -z[..., None]], -1).reshape(-1, 3).astype(np.float32)
    idx = np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)
    col = rng.integers(0, 256, (len(pos), 3)).astype(np.uint8)
    uv = rng.uniform(-2, 2, (len(pos), 2)).astype(np.float32)
    uv[::7] = 0.0
    tex = rng.integers(0, 256, (16, 32, 3)).astype(np.uint8)
    kw = dict(uvs=uv, texture=tex) if textured else {}
    sc = ctx.upload(pos, col, idx, **kw)
    sn = ctx.sensor(64, 64, 90.0, 1.0)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    want = oracle.render_view(pos, col, idx, 64, 64, pose[0], near_m=1.0, **kw)
    for ts in (0, 8, 16, 32):
        o = ctx.alloc(sn, 1, tri=True)
        ctx.render(sc, sn, pose, out=o, tile_size=ts)
        g = to_np(o)
        assert (g["tri"][0] == want["tri"]).all(), ts
        assert np.abs(g["rgb"][0].astype(int) - want["rgb"].astype(int)).max() <= 1, ts
        assert np.abs(g["depth"][0] - want["depth"]).max() <= 1e-5 * max(1.0, float(want["depth"].max())), ts
    assert ctx.get_error() == 0
    ctx.release(sc)


@pytest.mark.parametrize("n", [8, 96, 120, 232])    # 295 bands a view: one, one, two and four a block
@pytest.mark.parametrize("textured", [False, True])
def test_blocks_of_several_bands(ctx, n, textured):
    import torch
    import paper_1904_01201_amd as P
    note(f"shading: {n} views, textured {textured}")
    room = configs.room_2k_128()
    scene = room.scenes[0]
    h = ctx.upload_scene(with_texture(scene, seed=4, size=256) if textured else scene)
    sn = ctx.sensor(131, 117, 90.0, 0.01, P.OUT_RGB | P.OUT_DEPTH | P.OUT_TRI | P.OUT_SEMANTIC)
    poses = np.tile(room.poses[:8, 0].reshape(8, 12), (n // 8 + 1, 1))[:n]
    one = ctx.alloc(sn, 8)
    ctx.render(h, sn, poses[:8], out=one, tile_size=8)
    many = ctx.alloc(sn, n)
    for t in many.values():
        t.fill_(77)
    ctx.render(h, sn, poses, out=many, tile_size=16, one_sequence=True)
    torch.cuda.synchronize()
    for k, t in many.items():
        for e in range(n):
            assert torch.equal(t[e], one[k][e % 8]), (k, e)
    assert ctx.get_error() == 0
    ctx.release(h)
