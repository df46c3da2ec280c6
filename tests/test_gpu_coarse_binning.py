"""Tile lists of triangles that touch many tiles: boxes on both sides of what one lane
walks, chunks of more survivors than a block holds in registers, views of up to and of
more tiles than are binned at once.  Bar: the oracle's triangles and work counters, and
the same bits in every tiling and through the overflow path."""
import numpy as np
import pytest

import oracle
from tests.geom import pose_at
from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def soup(n, seed, extent):
    """n triangles of the given extent before the camera, all in view."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(-6.0, -2.0, (n, 1))
    mid = np.concatenate([rng.uniform(-0.7, 0.7, (n, 2)) * -z, z], 1)
    pos = mid[:, None, :] + rng.uniform(-0.5, 0.5, (n, 3, 3)) * extent * np.array([1.0, 1.0, 0.1])
    return pos.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.uint32).reshape(n, 3)


@pytest.mark.parametrize("n,extent", [(1, 3.0), (63, 0.5), (2500, 1.5), (9000, 0.3)])
@pytest.mark.parametrize("w,h", [(16, 16), (203, 117), (512, 256), (800, 700)])
def test_lists(ctx, n, extent, w, h):
    import torch
    pos, idx = soup(n, n + w, extent)
    col = np.random.default_rng(1).integers(0, 256, (len(pos), 3)).astype(np.uint8)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(w, h, 90.0, 0.1)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    note(f"coarse binning: {n} triangles of {extent} m, {w}x{h}")
    want = oracle.render_view(pos, col, idx, w, h, pose[0], near_m=0.1)
    first = None
    for kw in (dict(tile_size=16), dict(tile_size=8), dict(tile_size=32), dict(tile_size=16, bin_factor=0.4),
               dict(tile_size=8, tile_cap=40), dict(tile_size=16, lane_owned_z=True), dict()):
        o = ctx.alloc(sn, 1, tri=True)
        for t in o.values():
            t.fill_(77)
        ctx.render(sc, sn, pose, out=o, stats=bool(kw), **kw)
        torch.cuda.synchronize()
        stats = o.pop("stats", None)
        assert (o["tri"].cpu().numpy().view(np.uint32)[0] == want["tri"]).all(), kw
        if stats:
            assert all(stats[0][k] == want["stats"][k] for k in stats[0]), (kw, stats, want["stats"])
        if first is None:
            first = o
        for k in o:
            assert torch.equal(o[k], first[k]), (kw, k)
    assert ctx.get_error() == 0
    ctx.release(sc)
