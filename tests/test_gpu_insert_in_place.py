"""Depth insertion with prob_out on the log-odds themselves: the probabilities of the result are left
there, as they are beside it."""

import numpy as np
import pytest

import oracle
from workloads import poses_ball
from workloads.configs import Camera

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(33, 20, 9), (40, 40, 40)], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("scans", [0, 1, 3])
def test_probabilities_in_place(dims, shift, scans):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    print(f"[gpu] insertion in place {dims} shift {shift} scans {scans}", flush=True)
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + scans)
    cam = Camera(24, 17, 80.0, 70.0, 3.0)
    poses = poses_ball(np.array(dims) * 0.05, 0.04 * min(dims), max(scans, 1), seed=4)[:scans]
    depth = rng.uniform(0.05, 3.5, size=(scans, 17, 24)).astype(np.float32)
    L0 = rng.uniform(-2.0, 3.0, size=(nz, ny, nx)).astype(np.float32)
    ctx = nbt.Context(0)
    m = nbt.Map(ctx, np.full((nz, ny, nx), 0.5, np.float32), 0.1, np.zeros(3, np.float32))
    L = torch.zeros(L0.size + shift, device="cuda")[shift:].view(L0.shape)
    L.copy_(torch.from_numpy(L0))
    nbt.insert_scans(m, cam, torch.from_numpy(poses).cuda(), torch.from_numpy(depth).cuda(), L, prob_out=L)
    torch.cuda.synchronize()
    ref = oracle.insert_scans((0.1, np.zeros(3, np.float32)), cam, poses, depth, L0) if scans else L0
    p = 1.0 / (1.0 + np.exp(-ref.astype(np.float64)))
    assert np.all(np.abs(L.cpu().numpy() - p) <= 4 * np.spacing(p.astype(np.float32)))
    assert not m._insert_ws.any()
    ctx.close()
