"""Launches whose descriptors travel as a kernel argument: around the number of views
that fit, against the tile lists (whose descriptors are copied), and captured:
replays draw the captured poses whatever the context rendered in between.  Bar:
the same bits."""
import numpy as np
import pytest

from scenegen import configs
from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 9])
@pytest.mark.parametrize("size", [(64, 48), (131, 117), (5, 3)])
def test_view_counts(ctx, n, size):
    import torch
    note(f"inline descriptors: {n} views of {size}")
    w = configs.room_2k_128()
    sc = ctx.upload_scene(w.scenes[0])
    sn = ctx.sensor(*size)
    poses = w.poses[:n, 0]
    ref = ctx.render(sc, sn, poses, out=ctx.alloc(sn, n, tri=True), tile_size=16)
    for _ in range(3):
        o = ctx.alloc(sn, n, tri=True)
        for t in o.values():
            t.fill_(77)
        ctx.render(sc, sn, poses, out=o)
        for k in o:
            assert torch.equal(o[k], ref[k]), k
    na = ctx.alloc(sn, n)
    ctx.render_noalloc(sc, sn, poses, na["rgb"], na["depth"])
    for k in na:
        assert torch.equal(na[k], ref[k]), k
    ctx.release(sc)


@pytest.mark.parametrize("n", [1, 4])
def test_captured(ctx, n):
    import torch
    note(f"inline descriptors captured: {n} views")
    w = configs.room_2k_128()
    sc = ctx.upload_scene(w.scenes[0])
    sn = ctx.sensor(96, 80)
    a, b = w.poses[:n, 0], w.poses[20:20 + n, 0]
    want = {}
    for name, p in (("a", a), ("b", b)):
        want[name] = ctx.alloc(sn, n)
        ctx.render_noalloc(sc, sn, p, want[name]["rgb"], want[name]["depth"])
    torch.cuda.synchronize()
    got = ctx.alloc(sn, n)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.render_noalloc(sc, sn, a, got["rgb"], got["depth"])
    for k in range(4):
        for t in got.values():
            t.fill_(k)
        other = ctx.alloc(sn, n)
        ctx.render_noalloc(sc, sn, b, other["rgb"], other["depth"])
        g.replay()
        torch.cuda.synchronize()
        for key in got:
            assert torch.equal(got[key], want["a"][key]), (k, key)
            assert torch.equal(other[key], want["b"][key]), (k, key)
    assert ctx.get_error() == 0
    ctx.release(sc)
