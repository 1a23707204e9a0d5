"""GPU checks of the codes over a map's life: words that grow with every update, more words than the
palette takes and few again, words kept from earlier updates, updates replayed from a captured graph with
new words in the grid, and maps of one, a few and many voxels on an axis, in every order.  The
walk by codes (the timed one) must visit the voxels of the walk by words, record by record."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nbt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    return nbt


def _grid(shape, values, seed, block=1):
    """Probabilities of `values` different values (occupied ones rare), equal in blocks."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    nx, ny, nz = shape
    small = [-(-n // block) for n in (nz, ny, nx)]
    p = 0.02 + 0.45 * torch.randint(0, values, small, device="cuda", generator=g) / values + 1e-3 * (seed % 7)
    p = torch.where(torch.rand(small, device="cuda", generator=g) < 0.02 / block, 0.5 + p, p)
    for a in range(3):
        p = p.repeat_interleave(block, a)
    p = p[:nz, :ny, :nx].float().contiguous()
    p[0, 0, 0], p[-1, -1, -1] = 0.0625 + 1e-4 * seed, 0.9375                 # met nowhere else
    return p


def _check(nbt, m, cam, poses, what):
    import torch
    got = nbt.trace_viewpoints(m, cam, poses)
    only, _ = nbt.eval_viewpoints(m, cam, poses, want_steps=False)
    ref = nbt.trace_rays(m, cam, poses)
    for k in ("hash", "gain", "steps", "stop_lin", "reason"):
        assert torch.equal(got[2][k], ref[k]), (what, k)
    mean = ref["gain"].sum(1) / ref["gain"].shape[1]
    assert torch.all((only.double() - mean).abs() <= 1e-6 * mean), what


def _poses(shape, voxel, n, seed):
    import torch
    from workloads import poses_ball
    c = np.array(shape) * voxel / 2
    return torch.from_numpy(poses_ball(c, 0.4 * min(shape) * voxel + 0.01, n, seed=seed)).cuda()


@pytest.mark.parametrize("layout", [0, 1, 2, 3], ids=["linear", "column4", "column2", "column8"])
def test_words_over_a_maps_life(nbt, layout):
    from workloads.configs import Camera
    shape, voxel = (118, 103, 97), 0.05
    cam, poses = Camera(70, 50, 90.0, 80.0, 6.0), _poses(shape, voxel, 8, 3)
    ctx = nbt.Context(0)
    ctx.set_map_layout(layout)
    m = nbt.Map(ctx, _grid(shape, 2, 1, 8), voxel, (0.0, 0.0, 0.0))
    # 16 updates apart the palette is gathered anew: an overflow ends there once few words are left
    lives = [2, 3, 5, 10, 20, 40, 70, 100, 150, 200, 221, 222, 223, 224, 240, 1000, 1000, 3, 3, 2, 500]
    for k, values in enumerate(lives + [3] * 16 + [30, 4000]):
        print(f"[gpu] update {k}: {values} values, layout {layout}", flush=True)
        m.update(_grid(shape, values, 10 + (k if k % 3 else 0), 1 if k % 2 else 8))
        m.check()
        _check(nbt, m, cam, poses, (k, values))
    ctx.close()


@pytest.mark.parametrize("shape", [(1, 1100, 1000), (3, 640, 600), (6, 500, 400), (9, 17, 7001 // 2), (17, 300, 260),
                                   (300, 17, 301), (301, 290, 13), (1100, 1000, 1), (62, 129, 200), (3000, 40, 12)],
                         ids=lambda s: "x".join(map(str, s)))
def test_shapes(nbt, shape):
    from workloads.configs import Camera
    cam, poses = Camera(31, 23, 100.0, 100.0, 500.0 if max(shape) > 2000 else 60.0), _poses(shape, 0.1, 12, 5)
    for layout in (0, 1, 2, 3):
        print(f"[gpu] codes of {shape}, layout {layout}", flush=True)
        ctx = nbt.Context(0)
        ctx.set_map_layout(layout)
        m = nbt.Map(ctx, _grid(shape, 2, 1, 4), 0.1, (0.0, 0.0, 0.0))
        for k, (values, block) in enumerate([(60, 1), (3, 8), (150, 3)]):
            m.update(_grid(shape, values, k, block))
            _check(nbt, m, cam, poses, (layout, values))
        ctx.close()


def test_replayed_updates(nbt):
    import torch
    from workloads.configs import Camera
    shape, voxel = (130, 110, 100), 0.05
    cam, poses = Camera(40, 30, 90.0, 80.0, 6.0), _poses(shape, voxel, 8, 3)
    ctx = nbt.Context(0)
    P = _grid(shape, 4, 1, 8)
    m = nbt.Map(ctx, P, voxel, (0.0, 0.0, 0.0))
    ig = torch.empty(8, device="cuda")
    nbt.eval_viewpoints(m, cam, poses, ig_out=ig, want_steps=False)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.update(P)
        nbt.eval_viewpoints(m, cam, poses, ig_out=ig, want_steps=False)
    for k, values in enumerate([4, 30, 5, 100, 600, 600, 3, 3]):
        print(f"[gpu] replay {k}: {values} values", flush=True)
        P.copy_(_grid(shape, values, k, 1 if k % 2 else 8))
        graph.replay()
        torch.cuda.synchronize()
        got = ig.clone()
        again, _ = nbt.eval_viewpoints(m, cam, poses, want_steps=False)
        assert torch.equal(got, again)
        _check(nbt, m, cam, poses, k)
    ctx.close()


def test_words_of_edge_hashes(nbt):
    """Words whose hash (times 0x9E3779B1) has lower 21 bits all ones or all zero, new in an update."""
    import torch
    from workloads.configs import Camera
    inv = pow(0x9E3779B1, -1, 2 ** 32)
    free, occupied = [], []
    for low in (0x1FFFFF, 0):
        w = np.array([inv * (h << 21 | low) % 2 ** 32 for h in range(2048)], np.uint32)
        gain = (w & np.uint32(0x7FFFFFFF)).view(np.float32)
        free += [p for p in gain[w < 2 ** 31] if 1e-3 < p < 0.5]
        occupied += [np.float32(1) - g for g in gain[w >= 2 ** 31] if 0.0 < g < 1.0 and
                     np.float32(1) - (np.float32(1) - g) == g and np.float32(1) - g > 0.15]
    assert len(free) >= 12 and len(occupied) >= 3
    shape, voxel = (118, 103, 97), 0.05
    cam, poses = Camera(70, 50, 90.0, 80.0, 6.0), _poses(shape, voxel, 8, 3)
    ctx = nbt.Context(0)
    for p, classify in [(p, (0.5, 0.5)) for p in free] + [(p, (0.15, 0.15)) for p in occupied]:
        print(f"[gpu] word of {p}, classified by {classify}", flush=True)
        P = torch.full(shape[::-1], 0.125, device="cuda")
        m = nbt.Map(ctx, P, voxel, (0.0, 0.0, 0.0), classify)
        assert m.info()["code_bytes"] > 0
        P[::9, ::7, ::5] = float(p)
        m.update(P)
        _check(nbt, m, cam, poses, p)
    ctx.close()
