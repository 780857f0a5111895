"""Prisms as far away as floats go beside ordinary ones (the sums that order a
view's entries then pass the largest float): no result changes."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Scene, make_c2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("near", [20, 3000])
def test_far_prisms_change_nothing(near):
    import torch
    w = make_c2(n_ground=3000, n_facade=0)
    mid = np.array([w.points.x.mean(), w.points.y.mean()])
    cen = np.add.reduceat(w.scene.xy.astype(np.float64), w.scene.vert_off[:-1], axis=0) / np.diff(w.scene.vert_off)[:, None]
    scene = w.scene.subset(np.sort(np.argsort(np.hypot(*(cen - mid).T))[:near]))
    sq = np.array([[0, 0], [1, 0], [1, 1], [0, 1]]) * 1e37
    far = np.concatenate([np.array(c) * 3e38 + sq * s for c in ((-1, -1), (1, -1), (-1, 1), (1, 1)) for s in (1, 0.5, 0.25)])
    off = np.concatenate([scene.vert_off, scene.vert_off[-1] + 4 * np.arange(1, 13)]).astype(np.int32)
    wide = Scene(off, np.concatenate([scene.xy, far.astype(np.float32)]),
                 np.concatenate([scene.height, np.full(12, 50.0, np.float32)]))
    ctx = sa.Context(0)
    path = sa.Path(ctx, sa.sunpath_for_span(w.span, 30.0))
    dp = sa.DevicePoints.from_workload(w.points)
    for mode in (sa.SA_ACCRUAL, sa.SA_SAMPLED):
        c0, m0, _ = sa.accumulate(ctx, sa.Scene.from_workload(ctx, scene), dp, path, mode)
        c1, m1, _ = sa.accumulate(ctx, sa.Scene.from_workload(ctx, wide), dp, path, mode)
        ctx.sync()
        assert c0.any()
        assert torch.equal(c0, c1)
        assert torch.allclose(m0, m1, rtol=1e-5, atol=1e-4)  # (spilled sets are added in no fixed order)
