"""Launches that are drawn without tile lists (checked: no count, scan or scatter
phase) in the forms that such a launch takes: mixed sizes, scenes, outputs, textures
and noise in one batch, two halves side by side, captured steps with host and device
poses, blocks of 16-, 32- and 64-pixel tiles unshared, and cluster lists longer than
a block holds at once.  Bar: the same bits as the tile lists, the oracle's triangles."""
import numpy as np
import pytest

import oracle
from scenegen import make_apartment, make_room, with_texture
from scenegen.walks import random_poses
from tests.geom import pose_at, unit_cube
from tests.gpu_common import compare, compare_noisy_depth, gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu
OUT = ("rgb", "depth", "tri", "semantic")


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def drawn(ctx, call):
    """(launch sequences, drawn without lists) of call()."""
    ctx.profile(True)
    ctx.profile_read()
    call()
    t = ctx.profile_read()
    ctx.profile(False)
    return t["reset"]["launches"], "bin_count" not in t


def _items(ctx, hs, sensors, poses, n, outs):
    got = []
    for k in range(n):
        sn = sensors[k % len(sensors)]
        o = ctx.alloc(sn, 1, tri=True)
        for t in o.values():
            t.fill_(77)
        outs.append(o)
        s = (k // 4) % len(hs)
        got.append((hs[s], sn, poses[s][k % len(poses[s])], *[o.get(x) for x in OUT], k))
    return got


def _same(a, b, what):
    import torch
    for k in a:
        assert torch.equal(a[k], b[k]), (what, k)


# fine triangles; tiny views in two halves; coarse triangles in images beyond the size limit of the others
@pytest.mark.parametrize("n,two", [(24, False), (1100, True), (12, False)])
def test_mixed_batch_and_captured_steps(ctx, n, two):
    import torch
    import paper_1904_01201_amd as P
    note(f"direct forms: {n} views")
    scs = [with_texture(make_apartment(seed=51, target_T=20_000, jitter_sigma=0.01), size=128) if n == 24 else
           with_texture(make_room(seed=52, num_boxes=1), size=64),
           make_apartment(seed=53, target_T=60_000, jitter_sigma=0.01) if n == 24 else
           make_room(seed=54, num_boxes=0 if n > 24 else 20)]
    hs = [ctx.upload_scene(s) for s in scs]
    sizes = {24: ((128, 128), (130, 97), (160, 120), (96, 64)), 1100: ((24, 20), (17, 9), (32, 12), (20, 24)),
             12: ((512, 512), (401, 333), (640, 481), (517, 300))}[n]
    sensors = [ctx.sensor(w, h, 90.0, 0.01, o, s) for (w, h), o, s in
               zip(sizes, (P.OUT_RGB | P.OUT_DEPTH, 11, P.OUT_DEPTH, P.OUT_RGB | P.OUT_DEPTH), (0.0, 0.0, 0.0, 0.1))]
    poses = [random_poses(s, 6, seed=55) for s in scs]
    ref, got = [], []
    ctx.render_batch(_items(ctx, hs, sensors, poses, n, ref), tile_size=16)
    its = _items(ctx, hs, sensors, poses, n, got)
    assert drawn(ctx, lambda: ctx.render_batch(its)) == (2 if two else 1, True)
    torch.cuda.synchronize()
    for k in range(n):
        _same(got[k], ref[k], ("batch", k))
    # the noise seed of step s is the view's plus s: the noisy views are compared in the first
    pz = np.stack([x[2] for x in its]).astype(np.float32).reshape(n, 12)
    dev = torch.from_numpy(pz).cuda()
    for what in ("host", "device"):
        st = ctx.stepper(its)
        for r in range(3):
            for o in got:
                for t in o.values():
                    t.fill_(77)
            if what == "host":
                st.step(pz)
            else:
                st.step_device(dev)
            torch.cuda.synchronize()
            for k in range(n):
                if r == 0 or k % 4 != 3:
                    _same(got[k], ref[k], (what, r, k))
        st.close()
    for k in (*range(8), n - 1):
        s, sn = scs[(k // 4) % 2], sensors[k % 4]
        tex = getattr(s, "texture", None)
        g = {x: v[0] for x, v in to_np(ref[k]).items()}
        o = oracle.render_view(s.positions, s.colors, s.indices, sn.width, sn.height, its[k][2], instances=s.instances,
                               uvs=None if tex is None else s.uvs, texture=tex, noise_sigma=sn.depth_noise_sigma,
                               noise_seed=k)
        if sn.depth_noise_sigma > 0:
            compare_noisy_depth(g.pop("depth"), o, sn.depth_noise_sigma, k)
        compare(g, o, k)
    assert ctx.get_error() == 0
    for h in hs:
        ctx.release(h)


# one cluster a view: tiles of 16 pixels (480 of them), 32 (768) and 64 (600), a block each
@pytest.mark.parametrize("n,w,h", [(40, 64, 48), (128, 64, 72), (600, 33, 20)])
def test_unshared_tiles(ctx, n, w, h):
    import torch
    pos, idx = unit_cube(-0.5, 0.5, -0.5, 0.5, -2.5, -1.5)
    sc = ctx.upload(pos, np.random.default_rng(2).integers(0, 256, (len(pos), 3)).astype(np.uint8), idx)
    rng = np.random.default_rng(3)
    poses = np.concatenate([pose_at(*p).reshape(1, 12) for p in rng.uniform(-0.6, 0.6, (n, 3))])
    note(f"direct forms: {n} views of {w}x{h}, a block per tile")
    sn = ctx.sensor(w, h)
    outs = [ctx.alloc(sn, n, tri=True) for _ in range(2)]
    for o in outs:
        for t in o.values():
            t.fill_(77)
    assert drawn(ctx, lambda: ctx.render(sc, sn, poses, out=outs[0])) == (1, True)
    ctx.render(sc, sn, poses, out=outs[1], tile_size=8)
    torch.cuda.synchronize()
    _same(*outs, (n, w, h))
    want = oracle.render_view(pos, np.zeros((len(pos), 3), np.uint8), idx, w, h, poses[n // 2])
    assert (to_np(outs[0])["tri"][n // 2] == want["tri"]).all()
    ctx.release(sc)


def test_cluster_lists_longer_than_a_block_holds(ctx):
    """Two million triangles, 31,250 clusters, 15 blocks a tile: a block looks through 1,500 clusters, more than it
    tests in a round; from far above its 2,083 all meet the tile, more than it lists at once."""
    import torch
    n = 1000
    g = np.linspace(0.0, 20.0, n + 1)
    x, z = np.meshgrid(g, g, indexing="ij")
    rng = np.random.default_rng(56)
    y = 0.5 + 0.3 * np.sin(1.3 * x) * np.cos(z) + rng.uniform(0, 0.01, x.shape)
    i = np.arange((n + 1) ** 2).reshape(n + 1, n + 1)
    idx = np.stack([np.stack([i[:-1, :-1], i[1:, :-1], i[1:, 1:]], -1), np.stack([i[:-1, :-1], i[1:, 1:], i[:-1, 1:]], -1)],
                   2).reshape(-1, 3)
    pos = np.stack([x, y, z], -1).reshape(-1, 3)
    sc = ctx.upload(pos, rng.integers(0, 256, pos.shape).astype(np.uint8), idx)
    sn = ctx.sensor(800, 600, 90.0, 0.5)

    def above(h):
        return np.array([[10.0, h, 10.0, 1, 0, 0, 0, 0, 1, 0, -1, 0]], np.float32)

    note("direct forms: two million triangles from above")
    o = [ctx.alloc(sn, 1, tri=True) for _ in range(2)]
    assert drawn(ctx, lambda: ctx.render(sc, sn, above(10.0), out=o[0])) == (1, True)
    ctx.render(sc, sn, above(10.0), out=o[1], tile_size=16)
    torch.cuda.synchronize()
    _same(*o, "near")
    # a captured step keeps the path it was made with
    st = ctx.stepper([(sc, sn, above(10.0)[0], o[0]["rgb"][0], o[0]["depth"][0], o[0]["tri"][0])])
    for h in (900.0, 60.0, 10.0):
        for t in o[0].values():
            t.fill_(77)
        st.step_device(torch.from_numpy(above(h)).cuda())
        ctx.render(sc, sn, above(h), out=o[1], tile_size=16)
        torch.cuda.synchronize()
        _same(*o, h)
    st.close()
    assert ctx.get_error() == 0
    ctx.release(sc)
