"""Views of the scene (groups of 32 prisms, groups of 64 groups, 64 of those a
test): prism counts around each edge, walked by tiles of neighbouring points
and by tiles of points from all over the scene.  The packet kernels walk the
binary hierarchy with the same predicate per (point, instant), so counts and
bits are equal; the accrual form's minutes keep to the oracle by the bars of
the other parity tests (mean 1e-3, at most 0.5 minutes)."""
import numpy as np
import pytest

import oracle
import paper_1907_04435_amd as sa
from workloads import Points, Scene, Span
from workloads.scenes import Day

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return sa.Context(0)


def boxes(n, rng):
    """n rectangles of 4 to 9 m on a 12 m lattice, heights 3 to 60 m."""
    side = int(np.ceil(np.sqrt(n)))
    at = np.sort(rng.choice(side * side, n, replace=False))
    c = np.stack([at % side, at // side], 1) * 12.0 + 6.0
    w = rng.uniform(2.0, 4.5, (n, 2))
    xy = c[:, None, :] + w[:, None, :] * np.array([[-1, -1], [1, -1], [1, 1], [-1, 1]])
    off = np.arange(0, 4 * n + 1, 4, dtype=np.int32)
    return Scene(off, xy.reshape(-1, 2).astype(np.float32), rng.uniform(3.0, 60.0, n).astype(np.float32)), side * 12.0


@pytest.mark.parametrize("n_b", [1, 31, 32, 33, 64, 65, 2047, 2048, 2049, 2081, 131072, 131073])
@pytest.mark.parametrize("spread", [False, True])
def test_counts_equal_the_binary_walk(ctx, n_b, spread):
    import torch
    rng = np.random.default_rng(n_b)
    scene, side = boxes(n_b, rng)
    n = 333
    lo, hi = (0.0, side) if spread else (0.5 * side, 0.5 * side + 15.0)
    x, y = rng.uniform(lo, hi, n), rng.uniform(lo, hi, n)
    zero = np.zeros(n, np.float32)
    pts = Points(x.astype(np.float32), y.astype(np.float32), rng.uniform(0.0, 4.0, n).astype(np.float32), zero, zero,
                 np.full(n, -1, np.int32))
    span = Span(40.7, -74.0, [Day(2019, 6, 21, -4.0, (340.0, 1220.0))], 4.0)
    path = sa.Path(ctx, sa.sunpath_for_span(span, 40.0))
    sc = sa.Scene.from_workload(ctx, scene)
    dp = sa.DevicePoints.from_workload(pts)
    got = []
    for inst in (0, 8):
        ctx.set_launch(sampled_instants_per_packet=inst)
        c, m, b = sa.accumulate(ctx, sc, dp, path, sa.SA_SAMPLED, want_bits=True)
        got.append([t.cpu().numpy() for t in (c, m, b)])
    ctx.set_launch()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][2], got[1][2])
    few = pts.take(np.arange(0, n, 15))
    acc = sa.accumulate(ctx, sc, dp, path, sa.SA_ACCRUAL)[1].cpu().numpy()[0][::15]
    d = np.abs(acc - oracle.continuous(scene, few, oracle.sun_path(span, 40.0))["minutes"][0])
    say(f"{n_b} prisms: mean {got[0][0].mean():.1f} instants, accrual off by at most {d.max():.1e} min")
    assert d.mean() <= 1e-3 and d.max() <= 0.5
