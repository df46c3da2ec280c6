"""The scan of the tile counts with blocks of 64, 256 and 1024 threads, chosen by the
launch's largest view: views at both sides of each size, alone and with smaller
ones, at 8-, 16- and 32-pixel tiles.  Bar: the same bits as each view alone."""
import numpy as np
import pytest

from scenegen import configs
from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu

# 16-pixel tiles: 1, 63, 64, 72, 256, 272, 1024, 1056, 2115
SIZES = [(16, 16), (336, 48), (128, 128), (144, 128), (256, 256), (272, 256), (512, 512), (528, 512), (720, 750)]


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


@pytest.mark.parametrize("largest", range(len(SIZES)))
@pytest.mark.parametrize("ts", [8, 16, 32])
def test_block_sizes(ctx, largest, ts):
    import torch
    note(f"scan: up to {SIZES[largest]}, {ts}-pixel tiles")
    w = configs.room_2k_128()
    sc = ctx.upload_scene(w.scenes[0])
    sizes = [SIZES[largest]] + SIZES[:largest + 1] + [SIZES[largest // 2]]
    items, ref = [], []
    for k, (W, H) in enumerate(sizes):
        sn = ctx.sensor(W, H)
        o, r = ctx.alloc(sn, 1, tri=True), ctx.alloc(sn, 1, tri=True)
        for t in o.values():
            t.fill_(77)
        pose = w.poses[3 * k, 0]
        ctx.render(sc, sn, pose.reshape(1, 12), out=r, tile_size=ts)
        items.append((sc, sn, pose, o["rgb"], o["depth"], o["tri"]))
        ref.append(r)
    ctx.render_batch(items, tile_size=ts, one_sequence=True)
    torch.cuda.synchronize()
    for it, r in zip(items, ref):
        for t, k in ((it[3], "rgb"), (it[4], "depth"), (it[5], "tri")):
            assert torch.equal(t, r[k]), (it[1].width, it[1].height, k)
    assert ctx.get_error() == 0
    ctx.release(sc)
