"""Batched variants in units of (tile, part): point counts around a tile,
variants without points, points of no variant, few and many tiles, against
the same scene edited and evaluated variant by variant.  Minutes are the same
FP64 sums grouped differently (1e-6 relative covers their rounding to float32
beside the spilled sets' float adds); counts are equal but where a sample
instant falls on a window's edge (1e-4 of them, the other batched test's bar)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import make_c2, subset_points

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    ctx = sa.Context(0)
    w = make_c2(n_ground=20_000, n_facade=20_000)
    path = sa.Path(ctx, sa.sunpath_for_span(w.span, 30.0))
    return ctx, w, path


@pytest.mark.parametrize("lens", [[1], [64, 0, 65], [0, 0, 7, 200, 1], [1000] * 9, [30_000, 33]])
@pytest.mark.parametrize("grid", [0, 1, 300])
def test_units(setup, lens, grid):
    import torch
    ctx, w, path = setup
    lead, trail = 5, 3  # points before the first variant's and after the last's
    off = lead + np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n, V, k = int(off[-1]) + trail, len(lens), 4
    rng = np.random.default_rng(n)
    pts = w.points.take(subset_points(w.points, n, 17))
    ids = np.stack([rng.choice(w.scene.n_b, k, replace=False) for _ in range(V)]).astype(np.int32)
    h = rng.uniform(3.0, 300.0, (V, k)).astype(np.float32)
    sc = sa.Scene.from_workload(ctx, w.scene)
    dp = sa.DevicePoints.from_workload(pts)
    c = torch.full((path.n_bins, n), 3, dtype=torch.int32, device="cuda")
    m = torch.full((path.n_bins, n), 2.0, device="cuda")
    sa.sa_accumulate_batched(ctx, sc, torch.from_numpy(ids).cuda(), torch.from_numpy(h).cuda(), dp,
                             torch.from_numpy(off).cuda(), path, c, m, flags=sa.SA_FLAG_ADD, grid_blocks=grid)
    ctx.sync()
    c, m = c.cpu().numpy() - 3, m.cpu().numpy().astype(np.float64) - 2.0
    for part in (slice(0, lead), slice(n - trail, n)):
        assert not c[:, part].any() and not m[:, part].any()
    for v in range(V):
        if lens[v] == 0:
            continue
        at = np.arange(off[v], off[v + 1])
        sc.set_heights(ids[v], h[v])
        cv, mv, _ = sa.accumulate(ctx, sc, sa.DevicePoints.from_workload(pts.take(at)), path, sa.SA_ACCRUAL)
        sc.set_heights(ids[v], w.scene.height[ids[v]])
        cv, mv = cv.cpu().numpy(), mv.cpu().numpy()
        np.testing.assert_allclose(m[:, at], mv, rtol=1e-6, atol=2e-4)  # atol: minutes were added to 2
        assert (c[:, at] != cv).mean() <= 1e-4
    say(f"{lens} grid {grid}: equal")
