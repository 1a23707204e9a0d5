"""GPU parity of small per-perspective calls, whose rays are walked in segments: step counts, IG and
the per-ray records of the traced instance against the CPU oracle and the plain walk, from one ray
to grids beside the workgroups' shares, in every map order, with rays that miss the map, end in
their first voxel, cross it whole, and poses whose rotation stretches the rays beyond the table."""

import numpy as np
import pytest

import oracle
from workloads import look_at, poses_ball, scene_spheres
from workloads.configs import Camera
from workloads.scenes import SceneMap

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nbt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    return nbt


def _check(nbt, ctx, sc, cam, poses):
    import torch
    m = nbt.Map(ctx, sc.P, sc.voxel, sc.origin)
    dp = torch.from_numpy(np.ascontiguousarray(poses, np.float32)).cuda()
    ig, steps = nbt.eval_viewpoints(m, cam, dp)
    only, _ = nbt.eval_viewpoints(m, cam, dp, want_steps=False)
    tig, tsteps, rec = nbt.trace_viewpoints(m, cam, dp)
    ref = nbt.trace_rays(m, cam, dp)
    torch.cuda.synchronize()
    ig_ref, steps_ref = oracle.eval_viewpoints(sc, cam, poses)
    assert np.array_equal(steps.cpu().numpy().view(np.uint64), steps_ref)
    ig, only = ig.cpu().numpy(), only.cpu().numpy()
    nan = np.isnan(ig_ref)
    for got in (ig, only):
        assert np.array_equal(np.isnan(got), nan)
        assert np.all(np.abs(got[~nan] - ig_ref[~nan]) <= 1e-5 * np.maximum(np.abs(ig_ref[~nan]), 1e-30))
    assert np.array_equal(tig.cpu().numpy(), ig, equal_nan=True)
    assert torch.equal(tsteps, steps)
    for k in ("hash", "steps", "stop_lin", "reason", "reserved"):
        assert torch.equal(rec[k], ref[k]), k
    g, gr = rec["gain"].cpu().numpy(), ref["gain"].cpu().numpy()
    assert np.array_equal(g, gr, equal_nan=True)


@pytest.mark.parametrize("layout", [0, 1, 2, 3], ids=["linear", "column4", "column2", "column8"])
@pytest.mark.parametrize("n,w,h,rng_m", [(1, 1, 1, 2.0), (3, 3, 2, 3.0), (2, 5, 4, 0.7), (7, 8, 8, 2.0), (5, 9, 7, 6.0),
                                         (4, 20, 1, 2.0), (40, 16, 16, 2.5), (1, 65, 33, 4.0), (1, 200, 160, 3.0)])
def test_small_calls(nbt, layout, n, w, h, rng_m):
    print(f"[gpu] segments n={n} {w}x{h} range={rng_m} layout={layout}", flush=True)
    sc = scene_spheres(n=(70, 64, 75), voxel=0.05, n_spheres=30, seed=90 + w, origin=(0.1, -0.2, 0.3))
    ctx = nbt.Context(0)
    ctx.set_map_layout(layout)
    _check(nbt, ctx, sc, Camera(w, h, 70.0, 55.0, rng_m), poses_ball(sc.poi, 1.2, n, seed=n + w))
    ctx.close()


def test_odd_rays(nbt):
    rng = np.random.default_rng(8)
    P = rng.choice(np.array([0.05, 0.2, 0.35, 0.5, 0.9], np.float32), size=(41, 90, 33), p=[0.1, 0.4, 0.15, 0.34, 0.01])
    sc = SceneMap(P=P, voxel=0.1, origin=np.zeros(3, np.float32), poi=np.array([1.65, 4.5, 2.05]))
    poses = poses_ball(sc.poi, 2.0, 12, seed=4)
    poses[1] = look_at(np.array([[-3.0, 4.5, 2.05]]), sc.poi)[0]               # enters from outside
    poses[2] = look_at(np.array([[-3.0, -4.0, 2.0]]), np.array([-9.0, -9.0, 2.0]))[0]   # misses
    poses[3, :9] = np.eye(3, dtype=np.float32).ravel()                         # axis-aligned, ties
    poses[3, 9:] = (1.6, 4.5, 2.0)
    poses[4, :9] *= 40.0                                                       # stretched rays
    poses[5, :9] *= 1e-4                                                       # rays within a voxel
    poses[6, 4] = np.nan
    poses[7, :9] *= 1e6
    ctx = nbt.Context(0)
    for w, h in ((1, 1), (3, 3), (11, 6)):
        print(f"[gpu] segments odd rays {w}x{h}", flush=True)
        _check(nbt, ctx, sc, Camera(w, h, 60.0, 45.0, 5.0), poses)
    one = SceneMap(P=np.full((1, 1, 1), 0.5, np.float32), voxel=0.1, origin=np.zeros(3, np.float32), poi=np.full(3, 0.05))
    _check(nbt, ctx, one, Camera(4, 4, 60.0, 45.0, 5.0), poses_ball(one.poi, 0.3, 5, seed=2))
    ctx.close()
