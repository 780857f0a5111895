"""A bin a day over 192 years for one point: more bins in pieces than a grid
has rows.  Equal to the same days asked 35,000 at a time (FP64 sums of the same
segments, grouped differently: 1e-6 relative after rounding to float; the point
lies among few prisms, so no set spills)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Scene
from workloads.scenes import Points

pytestmark = pytest.mark.gpu


def test_seventy_thousand_bins():
    sq = np.array([[0, 0], [10, 0], [10, 10], [0, 10]], np.float32)
    scene = Scene(np.array([0, 4, 8], np.int32), np.concatenate([sq, sq + np.float32(25)]), np.array([30, 40], np.float32))
    f = lambda v: np.full(1, v, np.float32)  # noqa: E731
    pts = Points(f(18.0), f(20.0), f(0.0), f(0.0), f(0.0), np.full(1, -1, np.int32))
    ctx = sa.Context(0)
    sc, dp = sa.Scene.from_workload(ctx, scene), sa.DevicePoints.from_workload(pts)

    def run(year, days):
        sp = sa.sa_sunpath(40.7, -74.0, -5.0, year, 1, 1, days, 480.0, 960.0, 480.0, 30.0)
        c, m, _ = sa.accumulate(ctx, sc, dp, sa.Path(ctx, sp), sa.SA_ACCRUAL)
        ctx.sync()
        return c.cpu().numpy(), m.cpu().numpy()

    years = 192
    days = sum(366 if y % 4 == 0 and (y % 100 or y % 400 == 0) else 365 for y in range(1901, 1901 + years))
    assert days > 1 << 16
    c, m = run(1901, days)
    assert m.any()
    half = sum(366 if y % 4 == 0 and (y % 100 or y % 400 == 0) else 365 for y in range(1901, 1997))
    for at, (cp, mp) in ((0, run(1901, half)), (half, run(1997, days - half))):
        np.testing.assert_array_equal(c[at:at + len(cp)], cp)
        np.testing.assert_allclose(m[at:at + len(mp)], mp, rtol=1e-6)
