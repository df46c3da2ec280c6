"""Device memory of scenes: what a scene holds, and the upload memory that the
context keeps between uploads (bounded, reused, given back)."""
import ctypes as C

import numpy as np
import pytest

import oracle
from scenegen import make_apartment, make_room, with_texture
from scenegen.walks import random_poses
from tests.gpu_common import compare, gpu_ctx, note, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def _live(ctx):
    n, b = C.c_uint64(), C.c_uint64()
    assert ctx.lib.hab_test_live_allocations(C.byref(n), C.byref(b)) == 0
    return n.value, b.value


@pytest.mark.parametrize("textured", [False, True])
@pytest.mark.parametrize("tri", [20_000, 200_000])
def test_bytes_of_a_scene(ctx, tri, textured):
    s = make_apartment(seed=31, target_T=tri, jitter_sigma=0.01)
    if textured:
        s = with_texture(s, size=256)
    T = len(s.indices)
    h = ctx.upload_scene(s)
    before = _live(ctx)
    h2 = ctx.upload_scene(s)            # the second works in the memory kept
    after = _live(ctx)
    # positions 36, three colours 12 or texture coordinates 24, instance 4, cluster boxes half a byte a triangle
    want = (36 + (24 if textured else 12) + 4) * T + 32 * ((T + 63) // 64) + (4 * 256 * 256 if textured else 0)
    note(f"scene memory: {T} triangles, {h.device_bytes} bytes")
    assert h.device_bytes == want
    assert after[1] - before[1] == want
    ctx.release(h)
    ctx.release(h2)
    assert _live(ctx)[1] == before[1] - want


def test_uploads_share_the_memory_kept(ctx):
    """Scenes of growing and shrinking size, with and without colours and textures, uploaded on two streams one
    right after another: each renders as the oracle does."""
    import torch
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    scenes = [make_room(seed=32), with_texture(make_apartment(seed=33, target_T=30_000), size=64),
              make_apartment(seed=34, target_T=60_000, jitter_sigma=0.01), make_room(seed=35),
              with_texture(make_room(seed=36), size=128)]
    hs = [ctx.upload_scene(s, stream=streams[k % 2]) for k, s in enumerate(scenes)]
    plain = ctx.upload(scenes[0].positions, None, scenes[0].indices, stream=streams[1])
    sn = ctx.sensor(120, 90)
    note("scene memory: shared upload memory")
    for s, h in list(zip(scenes, hs)) + [(scenes[0], plain)]:
        pose = random_poses(s, 1, seed=37)
        g = to_np(ctx.render(h, sn, pose, out=ctx.alloc(sn, 1, tri=True)))
        tex = getattr(s, "texture", None)
        col = np.full_like(s.colors, 255) if h is plain else s.colors
        o = oracle.render_view(s.positions, col, s.indices, 120, 90, pose[0], uvs=None if tex is None else s.uvs,
                               texture=tex)
        compare({k: v[0] for k, v in g.items()}, o, "shared upload memory")
    assert ctx.get_error() == 0
    for h in hs + [plain]:
        ctx.release(h)


def test_large_upload_memory_is_given_back(ctx):
    rng = np.random.default_rng(38)
    small = make_room(seed=32)
    ctx.release(ctx.upload_scene(small))
    base = _live(ctx)
    V = 6_000_000                        # 72 MB of positions
    h = ctx.upload(rng.uniform(-1, 1, (V, 3)).astype(np.float32), None, rng.integers(0, V, (1000, 3)).astype(np.uint32))
    note("scene memory: large upload")
    assert _live(ctx)[1] <= base[1] + h.device_bytes
    ctx.release(h)
    ctx.release(ctx.upload_scene(small))
    assert _live(ctx)[1] <= base[1] + (1 << 20)
