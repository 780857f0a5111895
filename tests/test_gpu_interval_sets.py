"""Occluded sets whose lanes hold different numbers of members: a wave
inserts an interval by the shortest code that fits all of its lanes (empty
sets, at most one member, more).  Poles on part of a ring of growing
density, seen by one to two tiles of points beside and among them, against
the oracle on the same great circles; the height adjoint of the same sets."""
import numpy as np
import pytest

import oracle
import paper_1907_04435_amd as sa
from workloads.scenes import _pts

from gpu_util import run_lib, say
from test_gpu_spill import SPAN, ring_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return sa.Context(0)


@pytest.mark.parametrize("every", [1, 2, 5, 12, 40])
@pytest.mark.parametrize("n", [64, 100])
def test_sets_of_mixed_size(ctx, every, n):
    ring = ring_scene(n=120, r=30.0, hw=0.4)
    scene = ring.subset(np.arange(0, 120, every))
    rng = np.random.default_rng(every)
    # inside the ring, in the open, and on a pole's roof-covered footprint
    x, y = rng.uniform(65, 135, n), rng.uniform(65, 135, n)
    x[0], y[0] = scene.footprint(0).mean(0)
    pts = _pts(x, y, np.full(n, 0.05))
    g = run_lib(ctx, scene, pts, SPAN, sa.SA_ACCRUAL, seg_min=60.0)
    path = oracle.sun_path(SPAN, 60.0)
    o = oracle.continuous(scene, pts, path)
    d = np.abs(g["minutes"] - o["minutes"])
    say(f"{scene.n_b} poles, {n} points: |A - D_L| mean {d.mean():.1e} max {d.max():.1e}")
    assert d.mean() <= 1e-3 and d.max() <= 0.01   # the accrual bar of the parity tests

    import torch
    p, sc = sa.Path(ctx, sa.sunpath_for_span(SPAN, 60.0)), sa.Scene.from_workload(ctx, scene)
    grad = torch.empty(scene.n_b, dtype=torch.float32, device="cuda")
    sa.sa_grad_heights(ctx, sc, sa.DevicePoints.from_workload(pts), p, None, grad)
    ctx.sync()
    ref = oracle.grad_implicit(scene, pts, path)
    err = np.abs(grad.cpu().numpy() - ref).max()
    say(f"  gradient |GPU - oracle| {err:.1e} of {np.abs(ref).max():.1e}")
    assert err <= 1e-3 * max(np.abs(ref).max(), 1.0)   # the adjoint's bar: 1e-3 of the largest entry
