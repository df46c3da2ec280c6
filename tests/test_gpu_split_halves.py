"""Batches that really are rendered as two launch sequences (checked: two resets a
call, twice the allocations of a captured step): work counters and outputs of every
view, host and device poses, and failing allocations of either half."""
import ctypes as C

import numpy as np
import pytest

from scenegen import make_apartment, make_room
from scenegen.walks import random_poses
from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu
KEYS = ("rgb", "depth", "tri")


def live(lib):
    n, b = C.c_uint64(), C.c_uint64()
    assert lib.hab_test_live_allocations(C.byref(n), C.byref(b)) == 0
    return n.value, b.value


@pytest.fixture(scope="module")
def ctx():
    c = gpu_ctx()
    yield c
    c.close()


def sequences(ctx, call):
    """Launch sequences that call() runs."""
    ctx.profile(True)
    ctx.profile_read()
    call()
    n = ctx.profile_read()["reset"]["launches"]
    ctx.profile(False)
    return n


# more views than are ever kept together; few large ones; many of middling size
@pytest.mark.parametrize("n,w,h", [(1101, 24, 20), (37, 500, 480), (121, 200, 160)])
def test_counters_outputs_and_poses(ctx, n, w, h):
    import torch
    note(f"split halves: {n} views of {w} x {h}")
    scenes = [make_room(seed=41), make_apartment(seed=42, target_T=20_000, jitter_sigma=0.01)]
    hs = [ctx.upload_scene(s) for s in scenes]
    poses = [random_poses(s, 5, seed=43) for s in scenes]
    sn = ctx.sensor(w, h)
    # view k: scene k % 2 (so the halves differ), one of five poses
    alone = {}
    for s in range(2):
        for p in range(5):
            alone[s, p] = ctx.render(hs[s], sn, poses[s][p], out=ctx.alloc(sn, 1, tri=True), tile_size=16, stats=True)
    of = [(k % 2, (k // 2) % 5) for k in range(n)]
    o = ctx.alloc(sn, n, tri=True)
    items = [(hs[s], sn, poses[s][p], *[o[x][k] for x in KEYS]) for k, (s, p) in enumerate(of)]

    def check(what, stats=None):
        torch.cuda.synchronize()
        for x in KEYS:
            ref = torch.cat([alone[q][x] for q in alone])
            index = torch.as_tensor([list(alone).index(q) for q in of], device="cuda")
            assert torch.equal(o[x], ref[index]), (what, x)
        if stats is not None:
            assert stats == [alone[q]["stats"][0] for q in of], what
        for t in o.values():
            t.fill_(77)

    got = []
    assert sequences(ctx, lambda: got.append(ctx.render_batch(items, stats=True))) == 2
    check("two sequences", got[0])
    assert sequences(ctx, lambda: got.append(ctx.render_batch(items, stats=True, one_sequence=True))) == 1
    check("one sequence", got[1])
    assert sequences(ctx, lambda: ctx.render_batch(items)) == 2
    check("two sequences, uncounted")
    pz = np.stack([poses[s][p] for s, p in of]).astype(np.float32).reshape(n, 12)
    before = live(ctx.lib)[0]
    one = ctx.stepper(items, one_sequence=True)
    single = live(ctx.lib)[0] - before
    one.close()
    st = ctx.stepper(items)
    assert live(ctx.lib)[0] - before == 2 * single
    dev = torch.from_numpy(pz).cuda()
    other = dev[torch.randperm(n, device="cuda")].contiguous()
    for r in range(3):
        st.step(pz)
        check(("host poses", r))
        st.step_device(other)
        st.step_device(dev)
        check(("device poses", r))
    st.close()
    assert ctx.get_error() == 0
    for h2 in hs:
        ctx.release(h2)


def _failing(lib, make, run):
    """run(ctx) with the k-th allocation failing, for every k it makes; the number of them."""
    import paper_1904_01201_amd as P
    for k in range(60):
        c = make()
        try:
            lib.hab_test_fail_alloc(k)
            try:
                run(c)
            except P.HabError as e:
                assert e.status == P.HAB_ERR_OUT_OF_MEMORY
                lib.hab_test_fail_alloc(-1)
                c.after(failed=True)
                continue
            lib.hab_test_fail_alloc(-1)
            c.after(failed=False)
            return k
        finally:
            lib.hab_test_fail_alloc(-1)
            c.ctx.close()
    raise AssertionError("never succeeded")


class _Case:
    def __init__(self, n, w, h, **kw):
        import torch
        self.ctx = gpu_ctx()
        s = make_room(seed=41)
        self.h, self.sn = self.ctx.upload_scene(s), self.ctx.sensor(w, h)
        self.poses = random_poses(s, n, seed=44)
        self.kw = kw
        self.out = self.ctx.alloc(self.sn, n, tri=True)
        ref = gpu_ctx()
        self.want = ref.render(ref.upload_scene(s), self.sn, self.poses, out=ref.alloc(self.sn, n, tri=True), tile_size=16)
        torch.cuda.synchronize()
        ref.close()
        self.held = live(self.ctx.lib)
        self.stepper = None

    def same(self):
        import torch
        torch.cuda.synchronize()
        for x in KEYS:
            assert torch.equal(self.out[x], self.want[x]), x

    def render(self):
        self.ctx.render(self.h, self.sn, self.poses, out=self.out, **self.kw)

    def capture(self):
        items = [(self.h, self.sn, self.poses[k], *[self.out[x][k] for x in KEYS]) for k in range(len(self.poses))]
        self.stepper = self.ctx.stepper(items, **self.kw)


class _Render(_Case):
    def after(self, failed):
        if failed:
            self.render()                     # the retry succeeds
        self.same()


class _Stepper(_Case):
    def after(self, failed):
        if failed:
            assert live(self.ctx.lib) == self.held
            self.capture()
        self.stepper.step(self.poses)
        self.same()
        self.stepper.close()
        assert live(self.ctx.lib) == self.held


@pytest.mark.parametrize("n,w,h", [(1101, 24, 20), (37, 500, 480)])
def test_failing_allocations_of_a_render(n, w, h):
    from paper_1904_01201_amd import binding as B
    lib = B.load()
    base = live(lib)
    note(f"split halves: failing allocations, {n} views of {w} x {h}")
    one = _failing(lib, lambda: _Render(n, w, h, one_sequence=True), lambda c: c.render())
    two = _failing(lib, lambda: _Render(n, w, h), lambda c: c.render())
    assert two > one >= 1, (one, two)         # the second half has a workspace of its own
    assert live(lib) == base


@pytest.mark.parametrize("n,kw", [(1101, {}), (33, dict(bin_factor=2.5))])
def test_failing_allocations_of_a_captured_step(n, kw):
    from paper_1904_01201_amd import binding as B
    lib = B.load()
    base = live(lib)
    note(f"split halves: failing allocations of a stepper, {n} views, {kw}")
    one = _failing(lib, lambda: _Stepper(n, 24, 20, one_sequence=True, **kw), lambda c: c.capture())
    two = _failing(lib, lambda: _Stepper(n, 24, 20, **kw), lambda c: c.capture())
    assert two == 2 * one >= 2, (one, two)
    assert live(lib) == base
