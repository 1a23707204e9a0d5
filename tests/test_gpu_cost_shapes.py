"""GPU check of the planner's cost terms at the edges of the kernel's split: horizons of one
state, exactly a workgroup's tile, one more than it and longer than a tile (their cost is then
summed by a launch of its own), and perspective counts below, at and beside the waves' shares,
the scalar-load blocks and the LDS chunks, with one horizon to a workgroup and with several, against the float64 reference."""

import math

import numpy as np
import pytest

from oracle import idw as I
from workloads import poses_ball, trajectories_walk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2.0, 0.7])
@pytest.mark.parametrize("h,k,nb,npp", [(1, 1, 1, 1), (7, 1, 2, 15), (3, 20, 1, 16), (5, 21, 3, 129), (2, 63, 17, 8),
                                        (3, 64, 2, 130), (2, 65, 2, 1025), (1, 100, 33, 7),
                                        (4, 32, 2, 1024), (2, 33, 2, 47), (3, 13, 2, 2500), (300, 60, 1, 40)])
def test_cost_terms_at_tile_edges(h, k, nb, npp, p):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    print(f"[gpu] cost terms h={h} k={k} nb={nb} np={npp} p={p}", flush=True)
    rng = np.random.default_rng(h * 1000 + k)
    poi = np.array([0.3, 0.4, 0.8], np.float32)
    id_pos = np.stack([poses_ball(poi, 1.0, npp, seed=70 + u)[:, 9:12] for u in range(nb)]).astype(np.float32)
    id_ig = rng.uniform(5.0, 60.0, size=(nb, npp)).astype(np.float32)
    poses = trajectories_walk(poi, h, k, seed=71).astype(np.float32)
    poses[h - 1, k - 1, 9:12] = id_pos[nb - 1, npp - 1]      # exactly on a perspective
    tan_h, tan_v = np.float32(math.tan(math.radians(60))), np.float32(math.tan(math.radians(60)))
    ctx = nbt.Context(0)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    G, O, cost = nbt.eval_cost(ctx, dev(id_pos), dev(id_ig), dev(poses), poi, tan_h, tan_v, p=p, w_i=25.0)
    torch.cuda.synchronize()
    for i in range(0, h, 1 + h // 20):
        g, o, c = I.horizon_cost(poses[i].astype(np.float64), poi.astype(np.float64), tan_h, tan_v,
                                 id_pos.astype(np.float64), id_ig.astype(np.float64), p=p, w_i=25.0)
        assert np.max(np.abs(G[i].cpu().numpy() - g) / g) <= 1e-5
        assert np.max(np.abs(O[i].cpu().numpy() - o)) <= 2e-6
        # cos within 2e-6 of at least cos 60 degrees, G within 1e-5: 25 / (O G + eps) within 2e-5
        assert abs(float(cost[i]) - c) <= 2e-5 * c
    ctx.close()
