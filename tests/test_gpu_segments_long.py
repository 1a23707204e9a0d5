"""GPU parity of small calls on maps so long that the segments' LDS table is near its limit: the timed
and the traced instance (which also holds the records there) against the oracle and the plain walk."""

import numpy as np
import pytest

from test_gpu_segments import _check, nbt  # noqa: F401
from workloads import look_at
from workloads.configs import Camera
from workloads.scenes import SceneMap

pytestmark = pytest.mark.gpu


# table blocks of 8 crossings for 64 rays: 75 to 81, 80 being the most that is kept
@pytest.mark.parametrize("side", [598, 606, 622, 630, 638, 646])
@pytest.mark.parametrize("n,w,h", [(1, 100, 80), (3, 64, 40), (2, 200, 1)])
def test_long_tables(nbt, side, n, w, h):  # noqa: F811
    print(f"[gpu] segments side {side} n={n} {w}x{h}", flush=True)
    rng = np.random.default_rng(side)
    P = rng.choice(np.array([0.05, 0.2, 0.5, 0.9], np.float32), size=(21, 26, side), p=[0.3, 0.4, 0.2995, 0.0005])
    sc = SceneMap(P=P, voxel=0.01, origin=np.zeros(3, np.float32), poi=np.array([side * 0.005, 0.13, 0.1]))
    pos = np.array([[0.02, 0.12, 0.1]]) + 0.01 * rng.uniform(size=(n, 3))
    ctx = nbt.Context(0)
    _check(nbt, ctx, sc, Camera(w, h, 2.0, 1.6, 9.0), look_at(pos, np.array([9.0, 0.13, 0.11])))
    ctx.close()
