"""The sampled form over more chunks of instants than one launch's mask words
hold (a year at one minute has 17,000): bins that go on in the next launch, and
longest runs cut between days, against the packet kernels, which need no masks.
All equal: the weights are halves and ones, whose sums below 2^23 are exact."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import make_c2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65, 16_385])
def test_year_of_minutes(n):
    import torch
    w = make_c2(n_ground=n, n_facade=0)
    mid = np.array([w.points.x.mean(), w.points.y.mean()])
    cen = np.add.reduceat(w.scene.xy.astype(np.float64), w.scene.vert_off[:-1], axis=0) / np.diff(w.scene.vert_off)[:, None]
    scene = w.scene.subset(np.sort(np.argsort(np.hypot(*(cen - mid).T))[:40]))
    sp = sa.sa_sunpath(40.7, -74.0, -5.0, 2019, 1, 1, 365, -1.0, -1.0, 1.0, 60.0)
    sp.day_bin = (np.arange(365) // 92).astype(np.int32)
    ctx = sa.Context(0)
    sc, path, dp = sa.Scene.from_workload(ctx, scene), sa.Path(ctx, sp), sa.DevicePoints.from_workload(w.points)
    got = []
    for packets in (0, 8):
        ctx.set_launch(sampled_instants_per_packet=packets)
        for longest in (False, True):
            c = torch.empty((4, n), dtype=torch.int32, device="cuda")
            m, L = torch.empty((4, n), device="cuda"), torch.zeros((4, n), device="cuda")
            sa.sa_accumulate(ctx, sc, dp, path, sa.SA_SAMPLED, c, m, longest=L if longest else None)
            ctx.sync()
            got.append((c, m, L))
    assert got[0][0].any()
    for a, b in zip(got[:2], got[2:]):
        for x, y in zip(a, b):
            assert torch.equal(x, y)
