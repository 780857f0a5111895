"""Scenes of more prisms than one block of the views holds (131,072): around
that number, several blocks, and more blocks than a wave has lanes (8.4M
prisms).  Against the scene of the prisms that can reach the points (the sun
stays above 15 degrees: at most 1,500 m), which has one block: counts and bit
vectors are equal; minutes are sums grouped differently where the order of the
walk decides what spills (1e-5); contributions and gradients are FP64 sums."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Scene
from workloads.scenes import Points

from gpu_util import say

pytestmark = pytest.mark.gpu

PITCH, REACH = 30.0, 1600.0


def city(n, seed=1):
    """n squares on a lattice, row by row, and the way to a part of them."""
    rng = np.random.default_rng(seed)
    k = int(np.ceil(np.sqrt(n)))
    i = np.arange(n)
    c = np.stack([(i % k) * PITCH, (i // k) * PITCH], 1).astype(np.float64)
    c += rng.uniform(-3, 3, c.shape)
    r = rng.uniform(6, 11, n)
    h = np.clip(20 * np.exp(rng.standard_normal(n)), 3, 400).astype(np.float32)

    def scene(ids):
        sq = np.array([[-1, -1], [1, -1], [1, 1], [-1, 1]])
        xy = (c[ids][:, None, :] + sq[None] * r[ids][:, None, None]).reshape(-1, 2).astype(np.float32)
        return Scene(np.arange(0, 4 * len(ids) + 1, 4, dtype=np.int32), xy, h[ids])

    return scene, c, k * PITCH


def points(at, seed):
    rng = np.random.default_rng(seed)
    x, y = (np.sort(rng.uniform(-40, 40, 900)) + a for a in at)  # along a diagonal, some on roofs
    z = np.where(rng.random(900) < 0.2, 25.0, 0.0)
    f = lambda a: a.astype(np.float32)  # noqa: E731
    zero = np.zeros(900, np.float32)
    return Points(f(x), f(y), f(z), zero, zero, np.full(900, -1, np.int32))


def results(ctx, scene, pts, path, want):
    import torch
    sc, dp = sa.Scene.from_workload(ctx, scene), sa.DevicePoints.from_workload(pts)
    out = {}
    c, m, _ = sa.accumulate(ctx, sc, dp, path, sa.SA_ACCRUAL)
    out["accrual counts"], out["accrual minutes"] = c, m
    c, m, b = sa.accumulate(ctx, sc, dp, path, sa.SA_SAMPLED, want_bits=True)
    out["sampled counts"], out["sampled minutes"], out["bits"] = c, m, b
    if want == "all":
        out["runs minutes"], out["longest minutes"] = sa.continuous_shadow(ctx, sc, dp, path, sa.SA_ACCRUAL)
        out["contribution"] = sa.building_contribution(ctx, sc, dp, path, torch.ones(dp.n, device="cuda"))
        g = torch.empty(scene.n_b, device="cuda")
        sa.sa_grad_heights(ctx, sc, dp, path, None, g)
        out["gradient"] = g[None]
        ids = torch.zeros((2, 0), dtype=torch.int32, device="cuda")
        c, m = torch.empty_like(out["accrual counts"]), torch.empty_like(out["accrual minutes"])
        sa.sa_accumulate_batched(ctx, sc, ids, ids.float(), dp, torch.tensor([0, 300, dp.n], device="cuda"), path, c, m)
        out["batched counts"], out["batched minutes"] = c, m
    ctx.sync()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("n,want", [(131_072, "all"), (131_073, "all"), (300_001, "all"), (8_450_000, "some")])
def test_as_without_the_far_prisms(n, want):
    ctx = sa.Context(0)
    path = sa.Path(ctx, sa.sa_sunpath(40.7, -74.0, -5.0, 2019, 3, 20, 2, 480.0, 960.0, 2.0, 30.0))
    scene, c, side = city(n)
    whole = scene(np.arange(n))
    for k, at in enumerate(((side / 2, side / 2), (side / 3, 100.0))):
        pts = points(at, k)
        ids = np.flatnonzero(np.abs(c - np.array(at)).max(1) < REACH)
        part = scene(ids)
        assert part.n_b <= 131_072
        a, b = results(ctx, whole, pts, path, want), results(ctx, part, pts, path, want)
        say(f"{n} prisms against {part.n_b} at {at}")
        assert a["accrual counts"].any()
        for name in a:
            x, y = a[name], b[name]
            if name in ("contribution", "gradient"):
                assert not np.delete(x, ids, axis=1).any()
                np.testing.assert_allclose(x[:, ids], y, rtol=1e-5, atol=1e-5 * np.abs(y).max())
            elif "minutes" in name:
                np.testing.assert_allclose(x, y, rtol=1e-5, atol=2e-4)
            else:
                np.testing.assert_array_equal(x, y)
