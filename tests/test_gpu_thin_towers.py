"""A city of thin towers, where one point-segment in 77 needs more than four
pieces: a call of four million points is answered, with the sums of the same
points asked in parts (counts equal; minutes of a spilled point are float sums
in no fixed order, 1e-5 relative).  And the adjoint: a quarter of a million
points in the ring of poles, of whose point-segments nearly every one spills,
against its parts (FP64 sums in no fixed order, rounded to float: 1e-5)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Scene
from workloads.scenes import Points

from gpu_util import say
from test_gpu_spill import CENTRE, SPAN, ring_scene

pytestmark = pytest.mark.gpu


def towers(k=100, pitch=6.0, hw=0.5):
    rng = np.random.default_rng(1)
    x, y = (a.ravel() + rng.uniform(-1.5, 1.5, k * k) for a in np.meshgrid(np.arange(k) * pitch, np.arange(k) * pitch))
    sq = np.array([[-hw, -hw], [hw, -hw], [hw, hw], [-hw, hw]])
    xy = (np.stack([x, y], 1)[:, None, :] + sq[None]).reshape(-1, 2).astype(np.float32)
    return Scene(np.arange(0, 4 * k * k + 1, 4, dtype=np.int32), xy, rng.uniform(15, 45, k * k).astype(np.float32))


def ground(x, y):
    x, y = x.astype(np.float32), y.astype(np.float32)
    z = np.zeros_like(x)
    return Points(x, y, z, z, z, np.full(len(x), -1, np.int32))


def test_four_million_points():
    import torch
    ctx = sa.Context(0)
    i = np.arange(1 << 22) % (1 << 16)  # 256 x 256 in Morton order, a metre apart, 64 times
    ix, iy = (sum(((i >> (2 * b + o)) & 1) << b for b in range(8)) for o in (0, 1))
    n = len(i)
    pts = ground(172.0 + ix, 172.0 + iy)
    sc = sa.Scene.from_workload(ctx, towers())
    path = sa.Path(ctx, sa.sa_sunpath(40.7, -74.0, -4.0, 2019, 3, 19, 4, -1.0, -1.0, 5.0, 30.0))
    work = torch.zeros(8, dtype=torch.int64, device="cuda")
    c = torch.empty((path.n_bins, n), dtype=torch.int32, device="cuda")
    m = torch.empty((path.n_bins, n), device="cuda")
    sa.sa_accumulate(ctx, sc, sa.DevicePoints.from_workload(pts), path, sa.SA_ACCRUAL, c, m, work=work)
    ctx.sync()  # raises where the queue overflowed
    say(f"{int(work[6])} of {int(work[5])} windows")
    assert int(work[6]) > 1 << 22
    step = 700_003
    for a in range(0, n, step):
        b = min(a + step, n)
        cp, mp, _ = sa.accumulate(ctx, sc, sa.DevicePoints.from_workload(pts.take(np.arange(a, b))), path, sa.SA_ACCRUAL)
        ctx.sync()
        assert torch.equal(cp, c[:, a:b])
        assert torch.allclose(mp, m[:, a:b], rtol=1e-5, atol=1e-4)


def test_adjoint_of_spilled_tiles():
    import torch
    ctx = sa.Context(0)
    rng = np.random.default_rng(6)
    n, scene = 250_000, ring_scene()
    pts = ground(CENTRE[0] + rng.uniform(-1, 1, n), CENTRE[1] + rng.uniform(-1, 1, n))
    sc, path = sa.Scene.from_workload(ctx, scene), sa.Path(ctx, sa.sunpath_for_span(SPAN, 30.0))

    def grad(p):
        g = torch.empty(scene.n_b, device="cuda")
        sa.sa_grad_heights(ctx, sc, sa.DevicePoints.from_workload(p), path, None, g)
        ctx.sync()
        return g.double().cpu().numpy()

    whole = grad(pts)
    parts = sum(grad(pts.take(np.arange(a, min(a + 70_001, n)))) for a in range(0, n, 70_001))
    np.testing.assert_allclose(whole, parts, rtol=1e-5, atol=1e-5 * np.abs(whole).max())
