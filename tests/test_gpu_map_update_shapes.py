"""GPU checks of the map update at the edges of its kernels: encoding of maps around the tile and
layer steps in every order (against the plain encoding of the linear order, rewritten by the
separate re-layout kernel), and depth insertion at image sizes beside the 16x16-pixel groups, voxel
counts that are no multiple of 8, arrays that are not 16-byte aligned, a map of more than 512
voxels on an axis, and rays along the axes and beside the map's faces (against the oracle)."""

import numpy as np
import pytest

import oracle
from workloads import look_at, poses_ball
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


def _scene(shape, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = shape
    P = rng.choice(np.array([0.0, 0.05, 0.2, 0.5, 0.9, 1.0], np.float32), size=(nz, ny, nx),
                   p=[0.05, 0.3, 0.3, 0.3, 0.04, 0.01])
    P += (P < 0.4) * rng.uniform(0, 0.05, size=P.shape).astype(np.float32)
    return SceneMap(P=P.astype(np.float32), voxel=0.1, origin=np.zeros(3, np.float32), poi=np.array(shape) * 0.05)


# 61..63 and 125..127: the padded side at and beside whole tiles and waves; the last two take 8 layers a thread
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 6, 3), (61, 5, 30), (62, 62, 6), (63, 9, 31), (127, 130, 33),
                                   (250, 222, 263), (319, 190, 197)], ids=lambda s: "x".join(map(str, s)))
def test_encoding(nbt, shape):
    import torch
    sc = _scene(shape, seed=shape[0])
    cam = Camera(40, 32, 70.0, 60.0, 40.0)
    poses = poses_ball(sc.poi, 0.4 * min(shape) * 0.1, 16, seed=3)
    dp = torch.from_numpy(poses).cuda()
    ctx = nbt.Context(0)
    ref = None
    other = torch.full(sc.P.shape, 0.5, device="cuda")
    for layout in (0, 1, 2, 3):
        print(f"[gpu] encoding {shape} layout {layout}", flush=True)
        ctx.set_map_layout(layout)
        m = nbt.Map(ctx, other, sc.voxel, sc.origin)
        m.update(torch.from_numpy(sc.P).cuda())
        m.check()
        m.set_layout((layout + 1) % 4)                       # every stored word goes through the re-layout
        got = nbt.trace_rays(m, cam, dp)
        if ref is None:
            ref = got
            want = oracle.trace_rays(sc, cam, poses)
            assert np.array_equal(got["hash"].cpu().numpy().reshape(-1).view(np.uint64), want["hash"].reshape(-1))
            assert np.array_equal(got["gain"].cpu().numpy().reshape(-1), want["gain"].reshape(-1))
        for k in ref:
            assert torch.equal(got[k], ref[k]), (layout, k)
        m.set_layout(layout)
        bad = sc.P.copy()
        bad[-1, -1, -1] = np.nan
        m.update(torch.from_numpy(bad).cuda())
        with pytest.raises(nbt.NbtError):
            m.check()
    ctx.close()


@pytest.mark.parametrize("shape,w,h", [((17, 19, 13), 1, 1), ((17, 19, 13), 16, 16), ((33, 20, 9), 17, 31),
                                       ((600, 21, 15), 33, 15), ((40, 41, 43), 50, 2)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("shift", [0, 1])
def test_insertion(nbt, shape, w, h, shift):
    import torch
    print(f"[gpu] insertion {shape} {w}x{h} shift {shift}", flush=True)
    sc = _scene(shape, seed=shape[1])
    rng = np.random.default_rng(w + h)
    cam = Camera(w, h, 80.0, 70.0, 6.0)
    poses = poses_ball(sc.poi, 0.045 * min(shape), 6, seed=5)
    poses[0, :9] = np.eye(3, dtype=np.float32).ravel()        # along an axis
    poses[1] = look_at(sc.poi[None], sc.poi + np.array([1.0, 0, 0]))[0]
    poses[2] = look_at(np.array([[-1.0, 0.7, 0.5]]), sc.poi)[0]      # from outside the map
    depth = rng.uniform(0.05, 7.0, size=(6, h, w)).astype(np.float32)
    depth[rng.random(depth.shape) < 0.2] = np.inf
    depth[rng.random(depth.shape) < 0.05] = np.nan
    L0 = rng.uniform(-2.5, 4.0, size=sc.P.shape).astype(np.float32)
    ctx = nbt.Context(0)
    m = nbt.Map(ctx, sc.P, sc.voxel, sc.origin)
    n = L0.size

    def placed(a):                                            # `shift` floats off a 16-byte boundary
        t = torch.zeros(n + shift, dtype=torch.float32, device="cuda")[shift:].view(sc.P.shape)
        t.copy_(torch.from_numpy(a))
        return t

    L, prob = placed(L0), placed(L0)
    nbt.insert_scans(m, cam, torch.from_numpy(poses).cuda(), torch.from_numpy(depth).cuda(), L, prob_out=prob)
    torch.cuda.synchronize()
    ref = oracle.insert_scans(sc, cam, poses, depth, L0)
    assert np.array_equal(L.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    p = 1.0 / (1.0 + np.exp(-ref.astype(np.float64)))
    assert np.all(np.abs(prob.cpu().numpy() - p) <= 4 * np.spacing(p.astype(np.float32)))
    assert int(m._insert_ws.abs().sum()) == 0
    ctx.close()
