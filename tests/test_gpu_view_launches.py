"""Every form over more segments than the views of one launch may take, by the
library's own sizes, bins cut by a launch's end among them.  The 21st of each
month on the block scene, a bin a day, against the same days one by one (a
launch each): counts and runs are equal; minutes are the same FP64 sums,
rounded to float once more where a launch ends (1e-6); contributions and
gradients are FP64 sums in no fixed order (gradients rounded to float once)."""
import datetime as dt
import os
import re

import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import Span, make_c2, subset_points
from workloads.scenes import Day, _nyc_tz

from gpu_util import say

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(sa.LIB_PATH), "csrc")


def constant(name, file):
    """The value of a constexpr of the library's sources."""
    text = open(os.path.join(CSRC, file)).read()
    return eval(re.search(rf"\b{name} = ([0-9l<> ]+);", text).group(1).replace("l", ""))


def view_bytes(n_b):
    n1 = -(-n_b // (1 << constant("kGroupBits", "sa_internal.h")))
    n2 = -(-n1 // (1 << constant("kSuperBits", "sa_internal.h")))
    assert 'sizeof(ViewEntry) == 32' in open(os.path.join(CSRC, "sa_internal.h")).read()
    return 32 * (n_b + (n1 if n1 > 1 else 0) + (n2 if n2 > 1 else 0))


def noalloc_bytes():
    text = open(os.path.join(os.path.dirname(CSRC), "..", "include", "shadow_accrual.h")).read()
    return eval(re.search(r"SA_NOALLOC_SCRATCH_BYTES \((.*?)\)", text).group(1).replace("ll", ""))


@pytest.fixture(scope="module")
def w():
    w = make_c2(n_ground=20_000, n_facade=20_000)
    idx = np.concatenate([subset_points(w.points.take(np.arange(20_000)), 1100, 31),
                          20_000 + subset_points(w.points.take(np.arange(20_000, 40_000)), 901, 32)])
    w.points = w.points.take(idx)
    return w


class Year:
    """The paths: all days and each on its own, at knots of `seg` minutes."""

    def __init__(self, w, seg):
        self.ctx = sa.Context(0)
        self.sc = sa.Scene.from_workload(self.ctx, w.scene)
        self.dp = sa.DevicePoints.from_workload(w.points)
        days = [dt.date(2019, m, 21) for m in range(1, 13)]
        days = [Day(d.year, d.month, d.day, _nyc_tz(d)) for d in days]
        spans = [Span(40.7, -74.0, d, 1.0) for d in [days] + [[d] for d in days]]
        self.whole, *self.days = (sa.Path(self.ctx, sa.sunpath_for_span(s, seg)) for s in spans)

    def both(self, run):
        """Results over the whole path, and the days' one after the other, as numpy."""
        whole = run(self.whole)
        parts = [run(p) for p in self.days]
        self.ctx.sync()
        host = lambda a: a.cpu().numpy().astype(np.float64)  # noqa: E731
        return [host(a) for a in whole], [np.concatenate([host(p[k]) for p in parts]) for k in range(len(whole))]


def test_views_of_one_launch_do_not_hold_the_year(w):
    y = Year(w, 5.0)
    per = constant("kViewBytes", "accumulate.hip") // view_bytes(w.scene.n_b)
    say(f"{y.whole.n_segments} segments, {per} a launch")
    assert per < y.whole.n_segments
    assert all(p.n_segments <= per for p in y.days)


def test_batched(w):
    import torch
    y = Year(w, 5.0)
    rng = np.random.default_rng(4)
    n, V, k = y.dp.n, 3, 6
    ids = torch.from_numpy(np.stack([rng.choice(w.scene.n_b, k, replace=False) for _ in range(V)]).astype(np.int32)).cuda()
    h = torch.from_numpy(rng.uniform(3.0, 300.0, (V, k)).astype(np.float32)).cuda()
    off = torch.tensor([0, 700, 1300, n], device="cuda")

    def run(path):
        c = torch.empty((path.n_bins, n), dtype=torch.int32, device="cuda")
        m = torch.empty((path.n_bins, n), device="cuda")
        sa.sa_accumulate_batched(y.ctx, y.sc, ids, h, y.dp, off, path, c, m)
        return c, m

    (c, m), (cd, md) = y.both(run)
    np.testing.assert_array_equal(c, cd)
    np.testing.assert_allclose(m, md, rtol=1e-6, atol=1e-4)


def test_longest(w):
    y = Year(w, 5.0)
    whole, days = y.both(lambda path: sa.continuous_shadow(y.ctx, y.sc, y.dp, path, sa.SA_ACCRUAL))
    for a, b in zip(whole, days):
        assert a.any()
        np.testing.assert_array_equal(a, b)


def test_contribution(w):
    import torch
    y = Year(w, 5.0)
    weight = torch.from_numpy(np.random.default_rng(2).uniform(0.5, 2.0, y.dp.n).astype(np.float32)).cuda()
    (a,), (b,) = y.both(lambda path: (sa.building_contribution(y.ctx, y.sc, y.dp, path, weight),))
    assert a.any()
    np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9 * b.max())


def test_gradient(w):
    import torch
    y = Year(w, 5.0)

    def run(path):
        g = torch.empty(w.scene.n_b, device="cuda")
        sa.sa_grad_heights(y.ctx, y.sc, y.dp, path, None, g)
        return (g[None],)

    (a,), (b,) = y.both(run)
    assert (a != 0).sum() > 100
    np.testing.assert_allclose(a[0], b.sum(0), rtol=1e-5, atol=1e-6 * np.abs(b).max())


@pytest.mark.parametrize("longest", [False, True])
def test_noalloc(w, longest):
    """A launch of the allocation-free call ends inside a day (with the
    longest runs, between days)."""
    import torch
    y = Year(w, 30.0)
    per, starts = noalloc_bytes() // view_bytes(w.scene.n_b), np.cumsum([p.n_segments for p in y.days])
    assert per < y.whole.n_segments and per not in starts
    n, out = y.dp.n, []
    for call in (sa.sa_accumulate, sa.sa_accumulate_noalloc):
        c = torch.empty((12, n), dtype=torch.int32, device="cuda")
        m, L = torch.empty((12, n), device="cuda"), torch.zeros((12, n), device="cuda")
        call(y.ctx, y.sc, y.dp, y.whole, sa.SA_ACCRUAL, c, m, longest=L if longest else None)
        y.ctx.sync()
        out.append((c, m, L))
    (c, m, L), (cn, mn, Ln) = out
    assert torch.equal(c, cn) and torch.equal(L, Ln)
    assert torch.allclose(m, mn, rtol=1e-6, atol=1e-4)
