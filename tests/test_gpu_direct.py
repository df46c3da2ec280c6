"""The direct path (draw.hip: no triangle lists; small default launches)
writes the same bits as the tile lists (an explicit tile size), in every
output, over the sizes where its rules change: triangles walked by a lane or
drawn by a wave, near-plane crossings, clusters dropped as hidden, tiles of 16,
32 and 64 pixels with and without shares, one view and many, odd image sizes
and several launch forms."""
import numpy as np
import pytest

import oracle
from scenegen import make_apartment, make_room, with_texture
from scenegen.walks import random_poses
from tests.geom import pose_at, quad, unit_cube
from tests.gpu_common import gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu
OUT = ("rgb", "depth", "tri", "semantic")


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def _same(a, b, what):
    import torch
    for k in a:
        assert torch.equal(a[k], b[k]), f"{what}: {k}"


def _both(ctx, sc, sn, poses, what):
    import torch
    outs = []
    for ts in (0, 8):
        o = ctx.alloc(sn, len(poses), tri=True)
        for t in o.values():
            t.fill_(77)
        ctx.render(sc, sn, poses, out=o, tile_size=ts)
        outs.append(o)
    torch.cuda.synchronize()
    _same(*outs, what)
    assert ctx.get_error() == 0
    return outs[0]


def _patch(n, size, z, seed, tilt=0.0):
    """A jittered n x n grid of quads of edge size at depth z, in random triangle order."""
    rng = np.random.default_rng(seed)
    g = np.arange(n + 1) * size - n * size / 2
    x, y = np.meshgrid(g, g, indexing="ij")
    p = np.stack([x, y, -z + tilt * x], -1).reshape(-1, 3) + rng.uniform(-0.2, 0.2, ((n + 1) ** 2, 3)) * size
    v = np.arange((n + 1) ** 2).reshape(n + 1, n + 1)
    a, b, c, d = (q.ravel() for q in (v[:-1, :-1], v[1:, :-1], v[1:, 1:], v[:-1, 1:]))
    t = np.concatenate([np.stack([a, b, c], 1), np.stack([a, c, d], 1)])
    return p.astype(np.float32), rng.permutation(t).astype(np.uint32)


# triangle edges in pixels at 256 px: below a pixel, around the lane walk's
# limits (boxes of 24, 48, 96 pixels), the wave's (1,024) and beyond
@pytest.mark.parametrize("px", [0.4, 3.0, 4.9, 7.0, 9.8, 14.0, 32.0, 45.0, 400.0])
def test_box_sizes(ctx, px):
    n = int(min(96, max(3, 300 / px)))
    size = px * 2.0 / 128.0                       # depth 2 m, focal length 128 px
    pos, idx = _patch(n, size, 2.0, 7, tilt=0.2)
    # a second surface behind the first, and coplanar duplicates
    p2, i2 = _patch(n, size * 1.7, 3.3, 8)
    pos = np.concatenate([pos, p2, pos])
    idx = np.concatenate([idx, i2 + (n + 1) ** 2, idx[: len(idx) // 2] + 2 * (n + 1) ** 2])
    sc = ctx.upload(pos, np.random.default_rng(1).integers(0, 256, (len(pos), 3)).astype(np.uint8), idx)
    poses = np.concatenate([pose_at(0, 0, 0).reshape(1, 12), pose_at(0.3, -0.2, -1.2).reshape(1, 12),
                            pose_at(0, 0, -1.99).reshape(1, 12)])
    note(f"direct: box size {px} px")
    o = _both(ctx, sc, ctx.sensor(256, 256), poses, px)
    want = oracle.render_view(pos, np.zeros((len(pos), 3), np.uint8), idx, 256, 256, poses[0])
    assert (to_np(o)["tri"][0] == want["tri"]).all()
    ctx.release(sc)


# scenes of 30k and 150k triangles: 32- and 64-pixel tiles, shared
@pytest.mark.parametrize("tri", [30_000, 150_000])
@pytest.mark.parametrize("w,h", [(1, 1), (3, 2), (33, 17), (64, 64), (203, 117), (1000, 37), (37, 1000), (800, 600)])
def test_image_sizes(ctx, w, h, tri):
    sc0 = make_apartment(seed=61, target_T=tri, jitter_sigma=0.01)
    sc = ctx.upload_scene(sc0)
    note(f"direct: {w}x{h}, {tri} triangles")
    _both(ctx, sc, ctx.sensor(w, h, 80.0), random_poses(sc0, 1 if w * h > 100_000 else 5, seed=62), (w, h))
    ctx.release(sc)


# few triangles in many views: a block per 16-, 32- and 64-pixel tile, unshared
@pytest.mark.parametrize("n,w,h", [(40, 64, 48), (150, 64, 64), (1100, 20, 12)])
def test_unshared_tiles(ctx, n, w, h):
    pos, idx = unit_cube(-0.5, 0.5, -0.5, 0.5, -2.5, -1.5)
    sc = ctx.upload(pos, np.random.default_rng(2).integers(0, 256, (len(pos), 3)).astype(np.uint8), idx)
    rng = np.random.default_rng(3)
    poses = np.concatenate([pose_at(*p).reshape(1, 12) for p in rng.uniform(-0.6, 0.6, (n, 3))])
    note(f"direct: {n} views of {w}x{h}")
    o = _both(ctx, sc, ctx.sensor(w, h), poses, (n, w, h))
    want = oracle.render_view(pos, np.zeros((len(pos), 3), np.uint8), idx, w, h, poses[n // 2])
    assert (to_np(o)["tri"][n // 2] == want["tri"]).all()
    ctx.release(sc)


@pytest.mark.parametrize("near", [0.01, 0.5, 2.5])
def test_near_plane_and_rotations(ctx, near):
    """Coarse room triangles across the near plane, from cameras that look anywhere."""
    sc0 = make_room(seed=63)
    sc = ctx.upload_scene(sc0)
    rng = np.random.default_rng(64)
    poses = random_poses(sc0, 40, seed=65)
    for p in poses:
        q, r = np.linalg.qr(rng.normal(size=(3, 3)))
        q = q * np.sign(np.diag(r))
        p[3:] = (q * np.sign(np.linalg.det(q))).astype(np.float32).ravel()
    note(f"direct: near {near}")
    _both(ctx, sc, ctx.sensor(160, 120, 100.0, near), poses, near)
    ctx.release(sc)


def test_every_output_and_launch_form(ctx):
    """A mixed batch, split and not, and a replayed stepper: every output, against the tile lists and the oracle."""
    import torch
    import paper_1904_01201_amd as P
    scs = [with_texture(make_apartment(seed=66 + k, target_T=t, jitter_sigma=0.01), size=256)
           for k, t in enumerate((60_000, 300_000))]
    hs = [ctx.upload_scene(s) for s in scs]
    sensors = [ctx.sensor(w, h, 90.0, 0.01, o, s) for w, h, o, s in
               ((128, 128, 3, 0.0), (130, 97, 11, 0.0), (160, 120, P.OUT_DEPTH, 0.0), (96, 64, 3, 0.1))]
    n = 24
    poses = [random_poses(s, n, seed=70 + k) for k, s in enumerate(scs)]

    def items(outs):
        got = []
        for k in range(n):
            sn = sensors[k % 4]
            o = ctx.alloc(sn, 1)
            for t in o.values():
                t.fill_(77)
            outs.append(o)
            got.append((hs[k % 2], sn, poses[k % 2][k], *[o.get(x) for x in OUT], k))
        return got

    ref = []
    ctx.render_batch(items(ref), tile_size=16)
    split = []   # 48 views: two halves side by side, each a direct launch
    ctx.render_batch(items(split) + items(split))
    torch.cuda.synchronize()
    for k in range(2 * n):
        _same(split[k], ref[k % n], ("split", k))
    for what, kw in (("batch", {}), ("stepper", None)):
        note(f"direct: mixed batch, {what}")
        got = []
        it = items(got)
        if kw is None:
            st = ctx.stepper(it)
            for _ in range(3):       # the noise seed of step s is the view's plus s: compare the first
                if _ == 1:
                    torch.cuda.synchronize()
                    keep = [{k: t.clone() for k, t in o.items()} for o in got]
                st.step(np.stack([x[2] for x in it]))
            torch.cuda.synchronize()
            for k in (k for k in range(n) if k % 4 != 3):
                _same(got[k], keep[k], ("replay", k))
            got = keep
            st.close()
        else:
            ctx.render_batch(it, **kw)
        torch.cuda.synchronize()
        for k in range(n):
            _same(got[k], ref[k], (what, k))
    for k in (1, 5, 20):
        o = oracle.render_view(scs[k % 2].positions, scs[k % 2].colors, scs[k % 2].indices,
                               *(lambda s: (s.width, s.height))(sensors[k % 4]), poses[k % 2][k])
        g = to_np(ref[k])
        if "tri" in g:
            assert (g["tri"][0] == o["tri"]).all()
    assert ctx.get_error() == 0
    for h in hs:
        ctx.release(h)


def test_occluder_at_equal_depth_keeps_the_tie_rule(ctx):
    """A cluster exactly as near as the surface in front of it is not hidden: the smaller index wins the tie."""
    p, i = quad([-2, -2, -3], [2, -2, -3], [2, 2, -3], [-2, 2, -3])
    # 200 copies of the same quad: 400 coplanar triangles, seven clusters
    pos = np.tile(np.asarray(p, np.float32).reshape(-1, 3), (200, 1))
    idx = (np.asarray(i, np.uint32).reshape(1, -1, 3) + 4 * np.arange(200, dtype=np.uint32)[:, None, None]).reshape(-1, 3)
    idx = idx[::-1].copy()
    sc = ctx.upload(pos, None, idx)
    sn = ctx.sensor(96, 96)
    o = _both(ctx, sc, sn, np.tile(pose_at(0, 0, 0).reshape(1, 12), (40, 1)), "ties")
    want = oracle.render_view(pos, np.full((len(pos), 3), 255, np.uint8), idx, 96, 96, pose_at(0, 0, 0))
    for k in (0, 39):
        assert (to_np(o)["tri"][k] == want["tri"]).all()
    ctx.release(sc)


def test_empty_scene_and_empty_view(ctx):
    pos, idx = quad([-1, -1, -2], [1, -1, -2], [1, 1, -2], [-1, 1, -2])
    empty = ctx.upload(pos, None, np.zeros((0, 3), np.uint32))
    behind = ctx.upload(pos, None, idx)
    sn = ctx.sensor(48, 40)
    for sc, z in ((empty, 0.0), (behind, -5.0)):
        o = _both(ctx, sc, sn, pose_at(0, 0, z).reshape(1, 12), "empty")
        g = to_np(o)
        assert (g["depth"] == 0).all() and (g["rgb"] == 0).all() and (g["tri"] == 0xFFFFFFFF).all()
        ctx.release(sc)
