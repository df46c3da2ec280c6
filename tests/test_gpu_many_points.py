"""Free-space queries over more points than one launch has threads for.  Bar: every
point's answer equals that of the same point in a small query."""
import numpy as np
import pytest

from tests.gpu_common import gpu_ctx, note

pytestmark = pytest.mark.gpu


def test_more_points_than_a_launch_takes():
    import torch
    n, m = (1 << 30) + 12_345, 1 << 20          # four lanes a point: 2^32 threads and more
    if not torch.cuda.is_available() or torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GiB of device memory")
    note(f"free space: {n} points")
    with gpu_ctx() as ctx:
        rng = np.random.default_rng(3)
        a = rng.uniform(0.0, 20.0, (300, 2))
        nav = ctx.nav_upload(np.concatenate([a, a + rng.uniform(-0.5, 0.5, (300, 2))], 1).astype(np.float32))
        few = torch.from_numpy(rng.uniform(-1.0, 21.0, (m, 2))).cuda()
        want = ctx.nav_free(nav, few, 0.3)
        assert 0 < int(want.sum()) < m
        pts = torch.empty((n, 2), dtype=torch.float64, device="cuda")
        for k in range(0, n, m):
            pts[k:k + m] = few[:min(m, n - k)]
        got = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        ctx.nav_free(nav, pts, 0.3, out=got)
        torch.cuda.synchronize()
        whole = n // m * m
        assert bool((got[:whole].view(-1, m) == want).all())
        assert torch.equal(got[whole:], want[:n - whole])
        del pts, got
        torch.cuda.empty_cache()
