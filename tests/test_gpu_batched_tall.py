"""A building without a roof (an infinite height) in one variant is that
variant's alone: the others' results are those of a call without it."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import make_c2

pytestmark = pytest.mark.gpu


def test_infinite_height_of_one_variant():
    import torch
    w = make_c2(n_ground=4000, n_facade=0)
    ctx = sa.Context(0)
    sc = sa.Scene.from_workload(ctx, w.scene)
    path = sa.Path(ctx, sa.sunpath_for_span(w.span, 30.0))
    n, V = w.points.n, 40
    # the buildings nearest the points, infinite in the first variant; the last one edits one far away
    mid = np.array([w.points.x.mean(), w.points.y.mean()])
    cen = np.add.reduceat(w.scene.xy.astype(np.float64), w.scene.vert_off[:-1], axis=0) / np.diff(w.scene.vert_off)[:, None]
    near = np.argsort(np.hypot(*(cen - mid).T))
    ids = torch.from_numpy(np.stack([near[:V], near[-V:]]).astype(np.int32)).cuda()
    off = torch.tensor([0, 64, n], device="cuda")
    dp = sa.DevicePoints.from_workload(w.points)
    got = []
    for tall in (np.inf, 30.0):
        h = torch.full((2, V), 30.0, device="cuda")
        h[0] = tall
        c = torch.empty((path.n_bins, n), dtype=torch.int32, device="cuda")
        m = torch.empty((path.n_bins, n), device="cuda")
        sa.sa_accumulate_batched(ctx, sc, ids, h, dp, off, path, c, m)
        ctx.sync()
        got.append((c[:, 64:].cpu().numpy(), m[:, 64:].cpu().numpy()))
    assert got[1][0].any()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    # sets that overflow are finished window by window, in the order the prisms come in
    np.testing.assert_allclose(got[0][1], got[1][1], rtol=1e-5, atol=1e-4)
