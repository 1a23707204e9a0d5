"""GPU parity of split union IG with boxes around a trajectory's share of the scratch (2^25 words
over the call's trajectories): all above it or some, led by workgroups of their own (up to four
trajectories a CU) or not, and boxes of
several LDS passes below it, shared by workgroups, against the CPU oracle."""

import numpy as np
import pytest

import oracle
from workloads import look_at, scene_spheres
from workloads.configs import Camera

pytestmark = pytest.mark.gpu


# shares of 2^25 / t words: 1.0, 2.0, 3.6 and 67 M positions; the map has 2.9 M
@pytest.mark.parametrize("t,waves", [(1100, 4), (536, 4), (300, 4), (16, 8)])
@pytest.mark.parametrize("layout", [0, 1], ids=["linear", "column4"])
def test_boxes_around_the_share(t, waves, layout):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    print(f"[gpu] large trajectory boxes t={t} waves={waves} layout={layout}", flush=True)
    sc = scene_spheres(n=(150, 140, 136), voxel=0.05, n_spheres=200, seed=79)
    cam = Camera(17, 16, 100, 100, 12.0)
    c = sc.poi
    aims = np.array([[1, 0, 0], [-1, 0.3, 0], [0, 1, 0], [0, -1, 0.2], [0.01, 0, 1], [0.01, 0.4, -1]])
    rng = np.random.default_rng(t)
    traj = np.empty((t, 6, 12), np.float32)
    for k in range(t):
        if k % 3 == 1:                                         # out of the map's corner: a small box
            traj[k] = look_at(0.4 + np.arange(6)[:, None] * 0.03 + np.zeros((6, 3)), np.full(3, -5.0))
        else:                                                  # every way: the whole map
            traj[k] = look_at(np.repeat((c + rng.uniform(-1, 1, 3))[None], 6, 0), c + 30 * aims)
    traj[2, 3, 10] = np.nan
    ctx = nbt.Context(0)
    ctx.set_traj_waves(waves)
    ctx.set_map_layout(layout)
    m = nbt.Map(ctx, sc.P, sc.voxel, sc.origin)
    ig, counts, visits = nbt.eval_trajectories(m, cam, torch.from_numpy(traj).cuda())
    torch.cuda.synchronize()
    ig_ref, counts_ref, visits_ref = oracle.eval_trajectories(sc, cam, traj)
    assert np.array_equal(counts.cpu().numpy().astype(np.uint32), counts_ref)
    assert np.array_equal(visits.cpu().numpy().view(np.uint64), visits_ref)
    ig = ig.cpu().numpy()
    assert np.array_equal(np.isnan(ig), np.isnan(ig_ref))
    ok = ~np.isnan(ig_ref)
    assert np.all(np.abs(ig[ok] - ig_ref[ok]) <= 1e-5 * np.abs(ig_ref[ok]))
    ctx.close()
