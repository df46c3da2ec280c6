"""Survivor slots of the setup's runs of four 64-triangle clusters: scenes that end
inside a run or a cluster, runs whose every triangle leaves two pieces (the slots
are full), clusters out of sight in between, lists that overflow (their tiles scan
all slots) and views of more tiles than the binning keeps in LDS.  Bar: the same
triangle ids, work counters and bits as the oracle's and as other tile sizes'."""
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


def _scene(n, seed, two_pieces, hide):
    """n triangles in front of the camera; two_pieces: one vertex behind the near plane at 1 m, so that clipping
    leaves a quad; hide: every third cluster lies behind the camera."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(2.0, 3.0, (n, 3))
    if two_pieces:
        z[:, 2] = rng.uniform(-0.5, 0.9, n)
    xy = (rng.uniform(-0.8, 0.8, (n, 1, 2)) + rng.uniform(-0.3, 0.3, (n, 3, 2))) * np.maximum(z, 1.0)[..., None]
    pos = np.concatenate([xy, -z[..., None]], -1)
    if hide:
        pos[np.arange(n) // 64 % 3 == 1] *= [1.0, 1.0, -1.0]
        pos[np.arange(n) // 64 % 3 == 1] += [0.0, 0.0, 2.0]
    return pos.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 320, 511, 1000, 2300])
@pytest.mark.parametrize("two_pieces", [False, True])
@pytest.mark.parametrize("hide", [False, True])
def test_slots_and_the_oracle(ctx, n, two_pieces, hide):
    import torch
    note(f"runs: {n} triangles, two pieces {two_pieces}, hidden clusters {hide}")
    pos, idx = _scene(n, n, two_pieces, hide)
    col = np.random.default_rng(1).integers(0, 256, (len(pos), 3)).astype(np.uint8)
    sc = ctx.upload(pos, col, idx)
    sn = ctx.sensor(72, 50, 90.0, 1.0)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    want = oracle.render_view(pos, col, idx, 72, 50, pose[0], near_m=1.0)
    first = None
    for ts in (16, 8, 32):
        for opts in ({}, {"tile_cap": 20}, {"bin_factor": 0.001}):
            o = ctx.alloc(sn, 1, tri=True)
            for t in o.values():
                t.fill_(77)
            got = ctx.render(sc, sn, pose, out=o, tile_size=ts, stats=True, **opts)
            assert (to_np(o)["tri"][0] == want["tri"]).all(), (ts, opts)
            if first is None:
                first = got
                assert got["stats"][0]["survivors"] == want["stats"]["survivors"]
            assert got["stats"] == first["stats"], (ts, opts)
            plain = ctx.alloc(sn, 1, tri=True)
            ctx.render(sc, sn, pose, out=plain, tile_size=ts, **opts)
            for k in plain:
                assert torch.equal(plain[k], first[k]), (ts, opts, k)
    assert ctx.get_error() == 0
    ctx.release(sc)


@pytest.mark.parametrize("size", [(720, 750), (740, 760)])   # 2115 16-pixel tiles: above what the binning keeps in LDS
def test_many_tiles(ctx, size):
    import torch
    note(f"runs: {size}")
    pos, idx = _scene(1500, 5, False, False)
    sc = ctx.upload(pos, None, idx)
    sn = ctx.sensor(size[0], size[1], 90.0, 1.0)
    pose = pose_at(0, 0, 0).reshape(1, 12)
    outs = []
    for ts in (8, 16, 32):
        o = ctx.alloc(sn, 1, tri=True)
        ctx.render(sc, sn, pose, out=o, tile_size=ts)
        outs.append(o)
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k], outs[0][k]), k
    want = oracle.render_view(pos, np.full((len(pos), 3), 255, np.uint8), idx, size[0], size[1], pose[0], near_m=1.0)
    assert (to_np(outs[0])["tri"][0] == want["tri"]).all()
    ctx.release(sc)
