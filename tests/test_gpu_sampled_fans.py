"""The sampled form by fans of instants against its packet kernels: the same
predicate per (point, instant), so counts and bit vectors are equal, and
minutes and longest runs equal up to the grouping of at most ~1,000 float
additions per bin of 0.5 to 60 minutes each (1e-6 relative)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Span, make_c2, subset_points
from workloads.scenes import Day, Scene, _pts

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return sa.Context(0)


@pytest.fixture(scope="module")
def block():
    return make_c2(n_ground=4000, n_facade=4000)


def both(ctx, scene, pts, sp, add=False):
    """Counts, minutes, longest and bits by fans and by packets."""
    import torch
    path = sa.Path(ctx, sp)
    sc = sa.Scene.from_workload(ctx, scene)
    dp = sa.DevicePoints.from_workload(pts)
    B, K = path.n_bins, path.n_samples
    got = {}
    for inst in (0, 8):
        ctx.set_launch(sampled_instants_per_packet=inst)
        outs = []
        for runs, bits in ((False, False), (True, False), (True, True)):
            c = torch.full((B, dp.n), 3, dtype=torch.int32, device="cuda")
            m = torch.full((B, dp.n), 5.0, device="cuda")
            L = torch.full((B, dp.n), 7.0, device="cuda") if runs else None
            b = torch.full(((K + 31) // 32, dp.n), -1, dtype=torch.int32, device="cuda") if bits else None
            sa.sa_accumulate(ctx, sc, dp, path, sa.SA_SAMPLED, c, m, b, flags=sa.SA_FLAG_ADD if add else 0,
                             out_scale=0.25, longest=L)
            ctx.sync()
            outs.append([None if t is None else t.cpu().numpy() for t in (c, m, L, b)])
        got[inst] = outs
    ctx.set_launch()
    for f, p in zip(got[0], got[8]):
        np.testing.assert_array_equal(f[0], p[0])
        np.testing.assert_allclose(f[1], p[1], rtol=1e-6, atol=1e-6)
        if f[2] is not None:
            np.testing.assert_allclose(f[2], p[2], rtol=1e-6, atol=1e-6)
        if f[3] is not None:
            np.testing.assert_array_equal(f[3], p[3])
    say(f"{len(pts.x)} points x {K} instants: equal, mean count {got[0][0][0].mean():.1f}")
    return got[0]


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1001])
@pytest.mark.parametrize("day_bin", [None, [0, 0, 0], [0, 1, 0]])
def test_fans_equal_packets(ctx, block, n, day_bin):
    span = Span(block.span.lat, block.span.lon, block.span.days, 1.0, day_bin)
    both(ctx, block.scene, block.points.take(subset_points(block.points, n, 5)), sa.sunpath_for_span(span, 30.0))


@pytest.mark.parametrize("step", [5.0, 15.0, 60.0])
def test_coarse_instants(ctx, block, step):
    """Chunks cut by the sun's arc; added to what the outputs hold."""
    days = [Day(2019, 6, 21, -4.0, (340.0, 1220.0)), Day(2019, 12, 21, -5.0, (481.0, 979.0))]
    span = Span(40.7, -74.0, days, step)
    both(ctx, block.scene, block.points.take(subset_points(block.points, 700, 6)), sa.sunpath_for_span(span, step),
         add=True)


def test_sun_through_the_zenith(ctx, block):
    """Equator, equinox: directions spread all round the zenith, fans without edges."""
    span = Span(0.0, 0.0, [Day(2019, 3, 20, 0.0, (700.0, 760.0))], 1.0)
    got = both(ctx, block.scene, block.points.take(subset_points(block.points, 900, 7)), sa.sunpath_for_span(span, 30.0))
    assert got[0][0].any()


def test_many_edges_and_edge_cases(ctx):
    """Footprints of 3 to 130 vertices (edges go 64 at a time), points inside
    them, on their roofs and above, one prism alone, no prism."""
    rng = np.random.default_rng(3)
    off, xy, h = [0], [], []
    for k, m in enumerate((3, 63, 64, 65, 130)):
        a = np.arange(m) * 2 * np.pi / m + 0.1 * k
        xy.append(np.stack([60.0 * k + 20 * np.cos(a), 30 * np.sin(a)], 1))
        off.append(off[-1] + m)
        h.append(20.0 + 15 * k)
    scene = Scene(np.array(off, np.int32), np.concatenate(xy).astype(np.float32), np.array(h, np.float32))
    x, y = rng.uniform(-60, 320, 2000), rng.uniform(-90, 90, 2000)
    pts = _pts(x, y, rng.choice([0.0, 5.0, 20.0, 35.0, 90.0], 2000))
    span = Span(40.7, -74.0, [Day(2019, 6, 21, -4.0, None)], 1.0)
    sp = sa.sunpath_for_span(span, 30.0)
    got = both(ctx, scene, pts, sp)
    assert got[0][0].max() == len(sp.t_min)   # inside a footprint: always
    both(ctx, scene.subset(np.array([2])), pts, sp)
    both(ctx, scene.subset(np.array([], np.int64)), pts, sp)


def test_several_launches(ctx, block):
    """More views than one launch holds (six days on 20,000 prisms), and more
    masks (a year on one prism, 20,000 points)."""
    days = [Day(2019, 6, 10 + d, -4.0, None) for d in range(6)]
    sp = sa.sunpath_for_span(Span(40.7, -74.0, days, 1.0, [0, 0, 1, 1, 1, 2]), 60.0)
    both(ctx, block.scene, block.points.take(subset_points(block.points, 300, 8)), sp)
    one = block.scene.subset(np.array([11]))
    c = one.centroids()[0]
    rng = np.random.default_rng(9)
    pts = _pts(c[0] + rng.uniform(-200, 200, 20000), c[1] + rng.uniform(-200, 200, 20000))
    sp = sa.sa_sunpath(40.7, -74.0, -5.0, 2019, 1, 1, 365, -1.0, -1.0, 1.0, 240.0)
    sp.day_bin = np.zeros(365, np.int32)
    both(ctx, one, pts, sp)
