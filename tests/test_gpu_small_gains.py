"""Per-perspective IG of maps whose gains are small (probabilities of 1e-9 to 1e-4), in calls whose
perspectives are shared by several workgroups: small ones walked in segments, larger ones by
single waves and by whole workgroups, the no-allocation variant and the batch.  A ray's gains
are summed in binary32 in runs of 8 (7 roundings, and one of each sum in binary64 to binary32), everything else in binary64 or finer:
relative error below 9 x 2^-24."""

import numpy as np
import pytest

import oracle
from workloads import poses_ball
from workloads.configs import Camera
from workloads.scenes import SceneMap

pytestmark = pytest.mark.gpu
TOL = 9 * 2.0 ** -24


@pytest.mark.parametrize("p", [1e-9, 1.5e-7, 1e-4])
@pytest.mark.parametrize("words", ["few", "many"])
@pytest.mark.parametrize("n,w,h", [(3, 9, 9), (1, 20, 20), (40, 24, 17), (2, 160, 120), (300, 64, 48)])
def test_small_gains(n, w, h, words, p):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    print(f"[gpu] small gains {words} {p} n={n} {w}x{h}", flush=True)
    rng = np.random.default_rng(n + w)
    shape = (110, 104, 121)
    P = np.full(shape, p, np.float32) if words == "few" else rng.uniform(0.5 * p, 2 * p, shape).astype(np.float32)
    sc = SceneMap(P=P, voxel=0.05, origin=np.zeros(3, np.float32), poi=np.array([3.0, 2.6, 2.7]))
    cam = Camera(w, h, 60.0, 45.0, 4.0)
    poses = poses_ball(sc.poi, 1.0, n, seed=n)
    ref, _ = oracle.eval_viewpoints(sc, cam, poses)
    ctx = nbt.Context(0)
    m = nbt.Map(ctx, P, sc.voxel, sc.origin)
    dp = torch.from_numpy(poses).cuda()
    got = {"eval": nbt.eval_viewpoints(m, cam, dp)[0], "ig only": nbt.eval_viewpoints(m, cam, dp, want_steps=False)[0],
           "noalloc": nbt.eval_viewpoints_noalloc(m, cam, dp, torch.empty(n, device="cuda"))[0]}
    b = nbt.Batch(ctx, [m], cam, n)
    got["batch"] = torch.empty(n, device="cuda")
    b.run(torch.tensor([0, n], dtype=torch.int32, device="cuda"), dp, got["batch"])
    torch.cuda.synchronize()
    for k, v in got.items():
        rel = np.abs(v.cpu().numpy().astype(np.float64) - ref) / ref
        assert rel.max() <= TOL, (k, rel.max())
    ctx.close()
