"""The raster maps build only texels that the points can read: a point's
counts must not depend on which other points are asked.  Points of one
corner, one point, a line and points around and far outside the city,
against the same points asked together with the whole city's (whose bounds
take every texel)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Span, make_c2
from workloads.scenes import _pts, concat_points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("texel", [1.5, 4.0])
@pytest.mark.parametrize("day", [1, 2])
def test_counts_do_not_depend_on_the_other_points(texel, day):
    w = make_c2(n_ground=1000, n_facade=0)
    keep = np.argsort(w.scene.centroids()[:, 1])[:700]     # the city's southern end
    scene = w.scene.subset(np.sort(keep))
    lo, hi = scene.xy.min(0), scene.xy.max(0)
    rng = np.random.default_rng(4)
    box = lambda n, x0, y0, x1, y1: _pts(rng.uniform(x0, x1, n), rng.uniform(y0, y1, n))  # noqa: E731
    sets = [box(500, lo[0], lo[1], lo[0] + 80, lo[1] + 60), box(1, *lo, *hi), box(65, lo[0], hi[1] - 40, hi[0], hi[1] - 40),
            box(300, lo[0] - 300, lo[1] - 300, lo[0] + 30, lo[1] + 30), box(100, hi[0] + 2e4, lo[1], hi[0] + 3e4, hi[1])]
    every = concat_points(sets + [box(2000, *lo, *hi), _pts(np.array([lo[0] - 5e3, hi[0] + 5e3]), np.array([lo[1] - 5e3, hi[1] + 5e3]))])
    d = w.span.days[day]
    path_of = lambda ctx: sa.Path(ctx, sa.sunpath_for_span(Span(w.span.lat, w.span.lon, [d], 1.0), 30.0))  # noqa: E731
    ctx = sa.Context(0)
    sc, path = sa.Scene.from_workload(ctx, scene), path_of(ctx)

    def ask(pts):
        c, m = sa.sam_accumulate(ctx, sc, sa.DevicePoints.ground_from_workload(pts), path, texel)
        ctx.sync()
        return c.cpu().numpy()[0], m.cpu().numpy()[0]

    call, mall = ask(every)
    assert call.sum() > 0
    at = 0
    for s in sets:
        c, m = ask(s)
        np.testing.assert_array_equal(c, call[at:at + s.n])
        np.testing.assert_array_equal(m, mall[at:at + s.n])
        at += s.n
