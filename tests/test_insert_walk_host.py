"""The mark walk of the depth insertion, built for the CPU with every store checked against the mark
array, against the oracle: cameras exactly on each face, edge and corner of the map, looking out,
in and along the faces, at +0 and -0 and a subnormal distance from a face, with returns and without;
cameras inside and outside; rays that only graze an edge."""

import ctypes as C
import importlib.util
import itertools
import os
import subprocess

import numpy as np
import pytest

import oracle
from workloads import look_at, poses_ball
from workloads.configs import Camera

HERE = os.path.dirname(os.path.abspath(__file__))
HIT, MISS, LMIN, LMAX = (np.float32(v) for v in oracle.DEFAULT_INSERT_PARAMS)


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    spec = importlib.util.spec_from_file_location("_walk_build", os.path.join(
        os.path.dirname(HERE), "paper_2503_22588_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    lib = str(tmp_path_factory.mktemp("walk") / "walk.so")
    cmd = [build.hipcc(), *build.COMMON, "--offload-host-only", "-shared", "-o", lib,
           os.path.join(HERE, "insert_walk_check.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    f = C.CDLL(lib).mark_scan
    f.restype = C.c_int64
    f.argtypes = [C.c_int] * 3 + [C.c_float, C.c_void_p, C.c_int, C.c_int, C.c_float, C.c_float, C.c_float,
                                  C.c_void_p, C.c_void_p, C.c_void_p]
    return f


def _check(walk, dims, voxel, origin, cam, poses, depth, what=""):
    nx, ny, nz = dims
    origin = np.ascontiguousarray(origin, np.float32)
    poses = np.ascontiguousarray(poses, np.float32)
    depth = np.ascontiguousarray(depth, np.float32)
    w, h, th, tv, far = cam.as_tuple()
    L0 = np.zeros((nz, ny, nx), np.float32)
    for k in range(len(poses)):
        marks = np.zeros((nz, ny, nx, 2), np.uint8)
        outside = walk(nx, ny, nz, voxel, origin.ctypes.data, w, h, th, tv, far, poses[k].ctypes.data,
                       depth[k].ctypes.data, marks.ctypes.data)
        assert outside == 0, (what, k, outside)
        got = np.where(marks[..., 1] > 0, HIT, np.where(marks[..., 0] > 0, MISS, np.float32(0)))
        ref = oracle.insert_scans((voxel, origin), cam, poses[k:k + 1], depth[k:k + 1], L0)
        assert np.array_equal(got, ref), (what, k, np.argwhere(got != ref)[:4])


def face_cameras(dims, voxel, eps=0.0):
    """Every position with each coordinate on the lower face, the upper face or inside, at least
    one on a face (moved by eps along it), looking along every axis and out of the map's centre."""
    top = np.array(dims) * voxel
    axes = [np.eye(3)[a] * s for a in range(3) for s in (1, -1)]
    out = []
    for at in itertools.product((0, 1, 2), repeat=3):
        if at == (1, 1, 1):
            continue
        pos = np.array([(eps, 0.37 * t, t + eps)[k] for k, t in zip(at, top)])
        for d in axes + [pos - top / 2, top / 2 - pos]:
            out.append(look_at(pos[None], pos + d)[0])
            out[-1][9:] = pos
    return np.array(out, np.float32)


@pytest.mark.parametrize("dims", [(16, 12, 20), (1, 5, 7), (8, 1, 1), (1, 1, 1), (600, 4, 3)],
                         ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("returns", [False, True], ids=["no return", "returns"])
def test_cameras_on_the_faces(walk, dims, returns):
    voxel = 0.125                            # coordinates on a face are exactly 0 or n
    poses = face_cameras(dims, voxel)
    rng = np.random.default_rng(sum(dims))
    for w, h in ((1, 1), (9, 7), (17, 3)):
        cam = Camera(w, h, 100.0, 90.0, 2.0)
        depth = rng.uniform(0.01, 2.5, size=(len(poses), h, w)) if returns else np.full((len(poses), h, w), np.inf)
        _check(walk, dims, voxel, np.zeros(3), cam, poses, depth, (w, h))


@pytest.mark.parametrize("eps", [-0.0, 1e-45, -1e-45, 3e-39, -3e-39, 1.2e-38, 1e-30, -1e-30])
def test_cameras_beside_the_faces(walk, eps):
    dims, voxel = (11, 9, 13), 0.125
    poses = face_cameras(dims, voxel, eps)
    if eps == 0.0:
        poses[:, 9:][poses[:, 9:] == 0] = np.float32(-0.0)
    cam = Camera(8, 8, 100.0, 90.0, 2.0)
    rng = np.random.default_rng(5)
    depth = np.where(rng.random((len(poses), 8, 8)) < 0.5, np.inf, rng.uniform(0.01, 2.5, size=(len(poses), 8, 8)))
    _check(walk, dims, voxel, np.zeros(3), cam, poses, depth)
    huge = poses.copy()
    huge[:, :9] *= np.float32(1e35)          # segments so long that the crossings are subnormal
    _check(walk, dims, voxel, np.zeros(3), cam, huge, depth)
    _check(walk, dims, voxel, np.zeros(3), cam, huge, np.full_like(depth, np.inf))


def test_faces_at_an_offset_origin(walk):
    dims, voxel, origin = (14, 10, 9), 0.25, np.array([-1.5, 2.0, 0.75])
    poses = face_cameras(dims, voxel)
    poses[:, 9:] += origin.astype(np.float32)
    cam = Camera(13, 11, 120.0, 110.0, 3.0)
    _check(walk, dims, voxel, origin, cam, poses, np.full((len(poses), 11, 13), np.inf))


def test_inside_outside_and_grazing(walk):
    dims, voxel = (40, 36, 44), 0.05
    ext = np.array(dims) * voxel
    rng = np.random.default_rng(9)
    poses = np.concatenate([poses_ball(ext / 2, 0.8, 20, seed=3), poses_ball(ext / 2, 6.0, 30, seed=4),
                            look_at(rng.uniform(-2, 4, size=(20, 3)), np.zeros(3)),
                            look_at(rng.uniform(-2, 4, size=(20, 3)), np.array([ext[0], 0, ext[2]]))])
    poses[3, :9] *= 50.0
    poses[5, :9] *= 1e-4
    poses[7, 4] = np.nan
    cam = Camera(24, 18, 80.0, 70.0, 5.0)
    depth = np.where(rng.random((len(poses), 18, 24)) < 0.5, np.inf, rng.uniform(0.0, 6.0, (len(poses), 18, 24)))
    _check(walk, dims, voxel, np.zeros(3), cam, poses, depth)
