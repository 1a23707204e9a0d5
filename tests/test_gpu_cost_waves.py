"""GPU check of the planner's cost terms in each form a call's sizes choose: 1, 2, 4, 8 and 16 waves
splitting a tile's perspectives (more and fewer distributions than waves, shares beside the scalar-load blocks and the
binary32 runs), one horizon to a workgroup at the rule's edges, against the float64 reference."""

import math

import numpy as np
import pytest

from oracle import idw as I
from workloads import poses_ball

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2.0, 1.3])
@pytest.mark.parametrize("h,k,nb,npp", [
    (3, 1, 1, 10), (70, 20, 1, 19), (9, 7, 19, 1),                         # one wave (and two: 19 pairs)
    (5, 3, 2, 11), (3, 65, 3, 13),                                         # two
    (9, 5, 3, 17), (300, 1, 1, 65), (2, 30, 41, 1),                        # four
    (5, 20, 1, 85), (64, 33, 13, 11),                                      # eight
    (40, 20, 2, 95), (1, 64, 33, 7), (257, 4, 8, 125), (20, 33, 9, 130),   # sixteen
    (256, 4, 8, 128), (384, 4, 8, 128), (7, 32, 1, 1000), (385, 4, 8, 128), (7, 20, 8, 124),  # one horizon a workgroup, and beside
    (12289, 40, 1, 85), (530000, 1, 1, 41), (530000, 1, 3, 5),             # four and fewer by the chip's size
])
def test_cost_terms(h, k, nb, npp, p):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    print(f"[gpu] cost waves h={h} k={k} nb={nb} np={npp} p={p}", flush=True)
    rng = np.random.default_rng(h + 31 * k)
    poi = np.array([0.3, 0.4, 0.8], np.float32)
    id_pos = np.stack([poses_ball(poi, 1.0, npp, seed=70 + u)[:, 9:12] for u in range(nb)]).astype(np.float32)
    id_ig = rng.uniform(5.0, 60.0, size=(nb, npp)).astype(np.float32)
    poses = poses_ball(poi, 1.2, h * k, seed=7).astype(np.float32).reshape(h, k, 12)
    poses[h - 1, k - 1, 9:12] = id_pos[nb - 1, npp - 1]      # exactly on a perspective
    poses[h // 2, 0, 9:12] = id_pos[0, 0]
    tan_h, tan_v = np.float32(math.tan(math.radians(60))), np.float32(math.tan(math.radians(60)))
    ctx = nbt.Context(0)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    G, O, cost = nbt.eval_cost(ctx, dev(id_pos), dev(id_ig), dev(poses), poi, tan_h, tan_v, p=p, w_i=25.0)
    G, O, cost = G.cpu().numpy(), O.cpu().numpy(), cost.cpu().numpy()
    for i in sorted({0, h // 2, h - 1, *range(0, h, 1 + h // 20)}):
        g, o, c = I.horizon_cost(poses[i].astype(np.float64), poi.astype(np.float64), tan_h, tan_v,
                                 id_pos.astype(np.float64), id_ig.astype(np.float64), p=p, w_i=25.0)
        assert np.max(np.abs(G[i] - g) / g) <= 1e-5
        assert np.max(np.abs(O[i] - o)) <= 2e-6
        # cos within 2e-6 of at least cos 60 degrees, G within 1e-5: 25 / (O G + eps) within 2e-5
        assert abs(float(cost[i]) - c) <= 2e-5 * c
    ctx.close()
