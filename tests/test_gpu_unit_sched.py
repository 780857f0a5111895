"""How a launch cuts its work into units changes speed only: results of point
counts around tiles, XCD ranges (eight tiles and a remainder) and one unit
per wave, under several launch sizes, against the same points inside one
large call.  Counts are equal; minutes and contributions are FP64 sums
grouped differently (1e-6 relative covers their rounding to float32)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import make_c2, subset_points

from gpu_util import say

pytestmark = pytest.mark.gpu

SIZES = [1, 64, 65, 7 * 64, 8 * 64 + 1, 9 * 64 - 1, 40 * 64 + 17]


@pytest.fixture(scope="module")
def setup():
    import torch
    ctx = sa.Context(0)
    w = make_c2(n_ground=20_000, n_facade=20_000)
    keep = np.sort(np.argsort(np.hypot(*(w.scene.centroids() - np.array([w.points.x.mean(), w.points.y.mean()])).T))[:3000])
    scene = w.scene.subset(keep)
    pts = w.points.take(subset_points(w.points, max(SIZES), 31))
    remap = np.full(w.scene.n_b, -1, np.int32)
    remap[keep] = np.arange(len(keep))
    pts.owner = np.where(pts.owner >= 0, remap[pts.owner], -1).astype(np.int32)
    path = sa.Path(ctx, sa.sunpath_for_span(w.span, 30.0))
    sc = sa.Scene.from_workload(ctx, scene)

    def ask(n, grid):
        ctx.set_launch(tile_grid_blocks=grid)
        dp = sa.DevicePoints.from_workload(pts.take(np.arange(n)))
        out = {}
        for mode in (sa.SA_ACCRUAL, sa.SA_SAMPLED):
            c, m, _ = sa.accumulate(ctx, sc, dp, path, mode)
            out[mode] = (c.cpu().numpy(), m.cpu().numpy())
        _, L = sa.continuous_shadow(ctx, sc, dp, path, sa.SA_ACCRUAL)
        out["longest"] = L.cpu().numpy()
        out["contribution"] = sa.building_contribution(ctx, sc, dp, path).sum(1).cpu().numpy()
        g = torch.empty(scene.n_b, dtype=torch.float32, device="cuda")
        sa.sa_grad_heights(ctx, sc, dp, path, None, g)
        out["grad"] = g.cpu().numpy()
        ctx.sync()
        ctx.set_launch()
        return out

    return ask, {}


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("grid", [0, 1, 8, 13, 512])
def test_units_do_not_change_results(setup, n, grid):
    ask, seen = setup
    if "all" not in seen:
        seen["all"] = ask(max(SIZES), 0)
    if n not in seen:
        seen[n] = ask(n, 0)
    ref, base, got = seen["all"], seen[n], ask(n, grid)
    for mode in (sa.SA_ACCRUAL, sa.SA_SAMPLED):
        np.testing.assert_array_equal(got[mode][0], ref[mode][0][:, :n])
        np.testing.assert_allclose(got[mode][1], ref[mode][1][:, :n], rtol=1e-6, atol=1e-5)
    np.testing.assert_allclose(got["longest"], ref["longest"][:, :n], rtol=1e-6, atol=1e-5)
    np.testing.assert_allclose(got["contribution"], base["contribution"], rtol=1e-6)
    np.testing.assert_allclose(got["grad"], base["grad"], rtol=1e-5, atol=1e-5 * np.abs(base["grad"]).max() + 1e-12)
    say(f"{n} points, {grid or 'resident'} blocks: equal")
