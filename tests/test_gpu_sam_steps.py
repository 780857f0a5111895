"""A segment's raster map is built while the one before is asked, in two maps by
turns, with prisms in groups of 1 to 16.  Paths of more segments than a map
word has stamps (255): the same call again, whose stamps wrap elsewhere, gives
the same counts.  Few and many prisms (group sizes follow their number):
splitting the path in two, hence other launches before and after each map,
gives counts that add up to the whole path's, and minutes to the rounding of
their sums (1e-6)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Span, make_c2
from workloads.scenes import Day, _pts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_b,step,seg", [(1, 20.0, 40.0), (17, 20.0, 40.0), (300, 5.0, 30.0), (2500, 10.0, 60.0), (33, 4.0, 4.0)])
def test_groups_and_stamps(n_b, step, seg):
    w = make_c2(n_ground=1000, n_facade=0)
    near = np.argsort(np.hypot(*(w.scene.centroids() - w.scene.centroids().mean(0)).T))[:n_b]
    scene = w.scene.subset(np.sort(near))
    lo, hi = scene.xy.min(0) - 20.0, scene.xy.max(0) + 40.0
    rng = np.random.default_rng(n_b)
    dp = sa.DevicePoints.ground_from_workload(_pts(rng.uniform(lo[0], hi[0], 700), rng.uniform(lo[1], hi[1], 700)))
    days = [Day(2019, 6, 21, -4.0, (480.0, 1080.0)), Day(2019, 9, 21, -4.0, (480.0, 1080.0))]
    ctx = sa.Context(0)
    sc = sa.Scene.from_workload(ctx, scene)

    def ask(days):
        path = sa.Path(ctx, sa.sunpath_for_span(Span(40.7, -74.0, days, step), seg))
        c, m = sa.sam_accumulate(ctx, sc, dp, path, 2.0)
        ctx.sync()
        return c.cpu().numpy(), m.cpu().numpy().astype(np.float64)

    whole, again, parts = ask(days), ask(days), [ask([d]) for d in days]
    np.testing.assert_array_equal(whole[0], again[0])
    np.testing.assert_array_equal(whole[1], again[1])
    np.testing.assert_array_equal(whole[0].sum(0), sum(p[0].sum(0) for p in parts))
    np.testing.assert_allclose(whole[1].sum(0), sum(p[1].sum(0) for p in parts), rtol=1e-6, atol=1e-4)
    assert whole[0].any()
