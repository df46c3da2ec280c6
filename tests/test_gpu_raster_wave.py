"""16-pixel tiles (a wave each) against 8-pixel tiles and the oracle, at the
sizes where their lists are cut: around one work item's entries, many items
merging into one tile, records of every form (packed, far vertices), more than
eight blocks a record, and the overflow path.  Bar: the same bits, and the same
work counters as the oracle."""
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


def _soup(n, size_px, spread_px, seed):
    """n triangles of about size_px, their centres within spread_px of pixel (24, 24) of a 64 x 64 view at depth 2-3 m."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(2.0, 3.0, n)
    c = 24.0 + rng.uniform(-spread_px, spread_px, (n, 2))
    p = c[:, None] + rng.uniform(-0.5, 0.5, (n, 3, 2)) * size_px
    xy = (p - 32.0) / 32.0 * z[:, None, None]
    pos = np.concatenate([xy * [1.0, -1.0], np.broadcast_to(-z[:, None, None], (n, 3, 1))], -1).reshape(-1, 3)
    return pos.astype(np.float32), np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)


# (triangles, their size, how far they spread): one to many work items in a tile
@pytest.mark.parametrize("n,size,spread", [(1, 3, 1), (64, 3, 4), (255, 3, 4), (256, 3, 4), (257, 3, 4), (512, 3, 4),
                                           (513, 4, 4), (5000, 4, 6), (300, 14, 8), (300, 40, 20), (200, 400, 20),
                                           (700, 9000, 30)])
@pytest.mark.parametrize("opts", [{}, {"tile_cap": 40}, {"bin_factor": 0.001}])
def test_list_lengths_and_record_forms(ctx, n, size, spread, opts):
    import torch
    note(f"raster wave: {n} triangles of {size} px, {opts}")
    pos, idx = _soup(n, size, spread, n + size)
    col = np.random.default_rng(4).integers(0, 256, (len(pos), 3)).astype(np.uint8)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(64, 64, 90.0, 1.0)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    outs = []
    for ts in (16, 8):
        o = ctx.alloc(sn, 1, tri=True)
        for t in o.values():
            t.fill_(77)
        outs.append(ctx.render(sc, sn, pose, out=o, tile_size=ts, stats=True, **opts))
    torch.cuda.synchronize()
    for k in ("rgb", "depth", "tri"):
        assert torch.equal(outs[0][k], outs[1][k]), k
    assert outs[0]["stats"] == outs[1]["stats"]
    want = oracle.render_view(pos, col, idx, 64, 64, pose[0], near_m=1.0)
    assert (to_np(outs[0])["tri"][0] == want["tri"]).all()
    # the same launch again, without counters and with stale keys in the scratch
    again = ctx.alloc(sn, 1, tri=True)
    ctx.render(sc, sn, pose, out=again, tile_size=16, **opts)
    for k in again:
        assert torch.equal(again[k], outs[0][k]), k
    assert ctx.get_error() == 0
    ctx.release(sc)
