"""Long height edits (staged in memory of the context) with region scores on
paths of more and more bins between them: nodes are those of a fresh upload."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import make_c2

pytestmark = pytest.mark.gpu


def test_edits_and_scores_in_turn():
    import torch
    w = make_c2(n_ground=500, n_facade=0)
    scene = w.scene.subset(np.arange(2000))
    ctx = sa.Context(0)
    sc = sa.Scene.from_workload(ctx, scene)
    rng = np.random.default_rng(3)
    off = torch.tensor([0, 100], dtype=torch.int64, device="cuda")
    for bins in (1, 3, 40):
        ids = rng.choice(2000, 900, replace=False).astype(np.int32)
        h = rng.uniform(5.0, 90.0, 900).astype(np.float32)
        sc.set_heights(ids, h)
        scene.height[ids] = h
        path = sa.Path(ctx, sa.sa_sunpath(40.7, -74.0, -5.0, 2019, 3, 1, bins, 600.0, 840.0, 30.0, 60.0))
        values = torch.ones((bins, 100), device="cuda")
        got = sa.shadow_score(ctx, path, values, np.full(bins, 240.0), off)
        ctx.sync()
        # every day spans 240 minutes: a fraction of 1 / 240 a bin and point, times 240
        np.testing.assert_allclose(got.cpu().numpy(), [100.0 * bins], rtol=1e-12)
        np.testing.assert_array_equal(sc.read_bvh()[0], sa.Scene.from_workload(ctx, scene).read_bvh()[0])
    del sc, path, ctx
    torch.cuda.synchronize()
