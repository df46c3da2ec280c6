"""Which launches are drawn without tile lists: those of small size whose work is
in proportion.  Checked by the phases that a call runs (count, scan and scatter
belong to the lists), by the outputs, and by the price against the lists."""
import numpy as np
import pytest

from scenegen import make_apartment, make_room
from scenegen.walks import random_poses
from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


@pytest.fixture(scope="module")
def scenes(ctx):
    """name -> (generated scene, its handle); *_sh: triangles in random order."""
    made = {"room": make_room(seed=11)}
    for t in (5_000, 9_700, 20_000, 60_000, 200_000, 1_000_000):
        made[f"apt{t}"] = make_apartment(seed=21, target_T=t, jitter_sigma=0.01)
    out = {k: (s, ctx.upload_scene(s)) for k, s in made.items()}
    for k, s in made.items():
        order = np.random.default_rng(3).permutation(len(s.indices))
        out[k + "_sh"] = (s, ctx.upload(s.positions, s.colors, s.indices[order]))
    yield out
    for _, h in out.values():
        ctx.release(h)


def far(y):
    """Looking straight down from above the middle of an apartment."""
    return np.array([[6.0, y, 6.0, 1, 0, 0, 0, 0, 1, 0, -1, 0]], np.float32)


# scene, views, width, height, height above (None: inside), drawn without lists
CASES = [
    ("room", 1, 128, 128, None, True), ("room", 1, 1000, 1000, None, True), ("room_sh", 3, 512, 512, None, True),
    ("apt20000", 1, 512, 512, None, True), ("apt60000", 1, 1000, 1000, None, True), ("apt60000", 8, 128, 128, None, True),
    ("apt200000", 1, 256, 256, None, True), ("apt200000", 16, 128, 128, None, True), ("apt1000000", 1, 512, 512, None, True),
    ("apt1000000", 1, 32, 24, None, True), ("apt200000_sh", 1, 128, 128, None, True), ("apt60000_sh", 4, 128, 128, None, True),
    ("apt1000000_sh", 1, 512, 512, None, False), ("apt1000000_sh", 1, 256, 256, None, False),
    ("apt200000_sh", 3, 512, 512, None, False), ("apt200000_sh", 16, 128, 128, None, False),
    ("apt60000_sh", 1, 512, 512, None, False), ("apt20000_sh", 1, 512, 512, None, False),
    ("apt60000", 1, 256, 256, 400.0, False), ("apt1000000", 1, 256, 256, 400.0, False), ("apt1000000", 1, 512, 512, 40.0, False),
    ("apt60000", 1, 256, 256, 8.0, True), ("room", 1, 128, 128, 40.0, True),
    # many pixels a triangle: larger launches too
    ("room", 5, 512, 512, None, True), ("room", 31, 256, 256, None, True), ("room", 16, 512, 512, None, True),
    ("room", 1, 2048, 2048, None, True), ("apt5000", 8, 512, 512, None, True), ("apt20000", 4, 512, 512, None, True),
    ("apt5000", 100, 128, 128, None, False), ("apt20000", 12, 512, 512, None, False), ("apt60000", 5, 512, 512, None, False),
    ("room", 5, 512, 512, 40.0, True), ("apt9700", 5, 512, 512, 40.0, False), ("apt20000", 4, 512, 512, 40.0, False),
    ("apt5000", 1, 2048, 2048, 400.0, True), ("apt9700_sh", 1, 128, 128, None, True), ("apt9700_sh", 4, 256, 256, None, True),
    ("apt9700_sh", 24, 256, 256, None, False),
    # fine triangles of at least a pixel
    ("apt20000", 8, 256, 256, None, True), ("apt20000", 12, 256, 256, None, False), ("apt60000", 4, 512, 512, None, False),
    # images that fill little of their tiles
    ("apt200000", 16, 129, 129, None, False), ("apt200000", 8, 129, 129, None, True), ("apt200000", 14, 200, 150, None, False)]


@pytest.mark.parametrize("scene,n,w,h,above,direct", CASES)
def test_choice_outputs_and_price(ctx, scenes, scene, n, w, h, above, direct):
    import torch
    s0, sc = scenes[scene]
    sn = ctx.sensor(w, h, 90.0, 0.01 if above is None and w <= 512 else 0.5 if w <= 1000 else 1.0)
    poses = random_poses(s0, n, seed=5) if above is None else np.repeat(far(above), n, 0)
    note(f"direct rule: {scene}, {n} of {w} x {h}, above {above}")
    outs = []
    for kw in (dict(), dict(tile_size=16)):
        o = ctx.alloc(sn, n, tri=True)
        for t in o.values():
            t.fill_(77)
        ctx.profile(True)
        ctx.profile_read()
        ctx.render(sc, sn, poses, out=o, **kw)
        phases = ctx.profile_read()
        ctx.profile(False)
        outs.append((o, "bin_count" not in phases))
    torch.cuda.synchronize()
    assert [d for _, d in outs] == [direct, False]
    for k in outs[0][0]:
        assert torch.equal(outs[0][0][k], outs[1][0][k]), k

    def us(**kw):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = 1e9
        for _ in range(12):
            a.record()
            ctx.render(sc, sn, poses, out=outs[0][0], **kw)
            b.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        return best

    # (the shuffled and far views took up to 7 times the lists' time)
    drawn, lists = us(), us(tile_size=16)
    note(f"direct rule: {drawn:.0f} us, lists {lists:.0f} us")
    assert drawn <= 1.35 * lists
    assert ctx.get_error() == 0
