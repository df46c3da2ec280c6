"""Batches on both sides of the rule that renders them as one or two launch
sequences: many small frames, few large ones, more views than are ever kept
together; eager, as a captured stepper and with halves forced off.  Bar: the same
bits as each view alone."""
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


# size / 2^20 of n views of W x H of a 2k-triangle room: n (W H + 500)
@pytest.mark.parametrize("n,W,H", [(31, 48, 40), (32, 48, 40), (33, 500, 480), (36, 500, 480), (80, 196, 196), (81, 194, 194),
                                   (81, 198, 198), (1024, 48, 40), (1025, 24, 20)])
def test_rule(ctx, n, W, H):
    import torch
    note(f"split: {n} views of {W} x {H}")
    w = configs.room_2k_128()
    sc = ctx.upload_scene(w.scenes[0])
    sn = ctx.sensor(W, H)
    poses = w.poses[:7, 0].reshape(7, 12)
    ref = ctx.alloc(sn, 7)
    for k in range(7):
        one = ctx.render(sc, sn, poses[k:k + 1], out=ctx.alloc(sn, 1), tile_size=16)
        for key in ref:
            ref[key][k] = one[key][0]
    pick = np.arange(n) % 7
    index = torch.as_tensor(pick, device="cuda")
    for one_sequence in (False, True):
        o = ctx.alloc(sn, n)
        for t in o.values():
            t.fill_(77)
        ctx.render(sc, sn, poses[pick], out=o, one_sequence=one_sequence)
        for key in o:
            assert torch.equal(o[key], ref[key][index]), (key, one_sequence)
    o = ctx.alloc(sn, n)
    st = ctx.stepper([(sc, sn, poses[0], o["rgb"][k], o["depth"][k], None) for k in range(n)])
    for _ in range(3):
        for t in o.values():
            t.fill_(77)
        st.step(poses[pick])
        torch.cuda.synchronize()
        for key in o:
            assert torch.equal(o[key], ref[key][index]), key
    st.close()
    assert ctx.get_error() == 0
    ctx.release(sc)
