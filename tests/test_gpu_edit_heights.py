"""Host height edits: up to 64 climb on their own, more refit the hierarchy;
either way nodes, and results, are those of a fresh upload."""
import numpy as np
import pytest

import paper_1907_04435_amd as sa
from workloads import make_c2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def city():
    return make_c2(n_ground=500, n_facade=0)


@pytest.mark.parametrize("n_b", [1, 2, 3, 65, 3000])
@pytest.mark.parametrize("k", [1, 2, 8, 64, 65, 1000])
def test_edit_equals_fresh_upload(city, n_b, k):
    if k > n_b and k > 2:
        k = n_b
    ctx = sa.Context(0)
    scene = city.scene.subset(np.arange(n_b))
    rng = np.random.default_rng(k)
    sc = sa.Scene.from_workload(ctx, scene)
    for turn in range(3):       # up, down, and neighbours in the hierarchy
        if turn < 2:
            ids = rng.choice(n_b, min(k, n_b), replace=False).astype(np.int32)
        else:
            order = sc.read_bvh()[1]
            at = rng.integers(0, n_b - min(k, n_b) + 1)
            ids = order[at:at + min(k, n_b)].astype(np.int32)
        h = (rng.uniform(300, 900, len(ids)) if turn == 0 else rng.uniform(3, 20, len(ids))).astype(np.float32)
        if turn == 1:           # one named twice keeps its last height
            ids, h = np.append(ids, ids[0]), np.append(h, np.float32(777.0))
        sc.set_heights(ids, h)
        scene.height[ids] = h   # in order: the last one stays
        fresh, order_f = sa.Scene.from_workload(ctx, scene).read_bvh()
        nodes, order_e = sc.read_bvh()
        np.testing.assert_array_equal(order_e, order_f)
        np.testing.assert_array_equal(nodes, fresh)
