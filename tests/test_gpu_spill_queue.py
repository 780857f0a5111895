"""More spilled point-segments in one launch than a million (the ring of
poles of the spill tests, every ground point near its centre asked at once): the
sums are those of the same points asked in parts.  Minutes of a spilled
point are float sums in no fixed order (1e-5 relative)."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads.scenes import Points

from gpu_util import say
from test_gpu_spill import CENTRE, SPAN, ring_scene

pytestmark = pytest.mark.gpu


def test_a_million_and_a_half_spilled_windows():
    import torch
    ctx = sa.Context(0)
    rng = np.random.default_rng(5)
    n = 250_000
    f = lambda a: a.astype(np.float32)  # noqa: E731
    zero = np.zeros(n, np.float32)
    pts = Points(f(CENTRE[0] + rng.uniform(-1, 1, n)), f(CENTRE[1] + rng.uniform(-1, 1, n)), zero, zero, zero,
                 np.full(n, -1, np.int32))
    sc, path = sa.Scene.from_workload(ctx, ring_scene()), sa.Path(ctx, sa.sunpath_for_span(SPAN, 30.0))
    work = torch.zeros(8, dtype=torch.int64, device="cuda")
    c = torch.empty((1, n), dtype=torch.int32, device="cuda")
    m = torch.empty((1, n), device="cuda")
    sa.sa_accumulate(ctx, sc, sa.DevicePoints.from_workload(pts), path, sa.SA_ACCRUAL, c, m, work=work)
    ctx.sync()  # raises where the queue overflowed
    say(f"{int(work[6])} windows")
    assert int(work[6]) > 1 << 20
    for a in range(0, n, 50_000):
        part = pts.take(np.arange(a, a + 50_000))
        cp, mp, _ = sa.accumulate(ctx, sc, sa.DevicePoints.from_workload(part), path, sa.SA_ACCRUAL)
        ctx.sync()
        assert torch.equal(cp, c[:, a:a + 50_000])
        assert torch.allclose(mp, m[:, a:a + 50_000], rtol=1e-5, atol=1e-4)
