"""GPU parity of union IG where one trajectory's rays are split over several workgroups and where
they are not: tile counts beside the split's steps, a non-finite pose in one of the trajectories,
bitsets covered in several passes, and a box larger than a trajectory's share of the scratch
(left to one workgroup) beside small ones, against the CPU oracle."""

import numpy as np
import pytest

import oracle
from workloads import look_at, scene_spheres, trajectories_walk
from workloads.configs import Camera

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nbt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    return nbt


def _compare(nbt, m, scene, cam, traj, want_visits=True):
    import torch
    ig, counts, visits = nbt.eval_trajectories(m, cam, torch.from_numpy(traj).cuda(), want_visits=want_visits)
    torch.cuda.synchronize()
    ig_ref, counts_ref, visits_ref = oracle.eval_trajectories(scene, cam, traj)
    assert np.array_equal(counts.cpu().numpy().astype(np.uint32), counts_ref)
    if want_visits:
        assert np.array_equal(visits.cpu().numpy().view(np.uint64), visits_ref)
    ig = ig.cpu().numpy()
    assert np.array_equal(np.isnan(ig), np.isnan(ig_ref))
    ok = ~np.isnan(ig_ref)
    assert np.all(np.abs(ig[ok] - ig_ref[ok]) <= 1e-5 * np.abs(ig_ref[ok]))
    return ig


# 8x8-pixel tiles x poses against 2 tiles for each of 4, 8 or 16 waves: 1 (unsplit), just below
# and at two workgroups, an odd number of them, and more tiles than divide evenly
@pytest.mark.parametrize("waves", [4, 8, 16])
@pytest.mark.parametrize("t,l,w,h", [(1, 1, 8, 8), (2, 15, 9, 8), (2, 31, 8, 8), (3, 32, 8, 8), (5, 7, 33, 17)])
def test_split_counts(nbt, waves, t, l, w, h):
    print(f"[gpu] split trajectories t={t} l={l} {w}x{h} waves={waves}", flush=True)
    sc = scene_spheres(n=(48, 40, 44), voxel=0.05, n_spheres=25, seed=77)
    cam = Camera(w, h, 60, 45, 1.0)
    traj = trajectories_walk(sc.poi, t, l, seed=5, r_range=(0.3, 0.6))
    if t > 2:
        traj[1, l // 2, 10] = np.nan
    ctx = nbt.Context(0)
    ctx.set_traj_waves(waves)
    m = nbt.Map(ctx, sc.P, sc.voxel, sc.origin)
    a = _compare(nbt, m, sc, cam, traj)
    b = _compare(nbt, m, sc, cam, traj, want_visits=False)
    assert np.array_equal(a, b, equal_nan=True)
    ctx.set_lds_budget(2048)                                   # several passes
    assert np.array_equal(a, _compare(nbt, m, sc, cam, traj), equal_nan=True)
    ctx.close()


def test_box_beyond_the_scratch(nbt):
    sc = scene_spheres(n=(150, 140, 136), voxel=0.05, n_spheres=200, seed=78)     # 2.9 M voxels
    cam = Camera(24, 24, 100, 100, 12.0)
    c = sc.poi
    every_way = look_at(np.repeat(c[None], 6, 0), c + np.array([[1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0],
                                                               [0.01, 0, 1], [0.01, 0, -1]]))
    corner = look_at(np.repeat((c * 0 + 0.4)[None], 6, 0) + np.arange(6)[:, None] * 0.03, np.full(3, -5.0))
    traj = np.stack([corner, every_way, corner[::-1]]).astype(np.float32)
    ctx = nbt.Context(0)
    m = nbt.Map(ctx, sc.P, sc.voxel, sc.origin)
    _compare(nbt, m, sc, cam, traj)
    ctx.close()
