"""What bench.py counts as gathered per voxel step (CPU only): a byte where the walk reads codes, a
word where it does not, in the rates, the fractions and the working set."""

import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402
from test_bench_helpers import CEIL  # noqa: E402

CODED = {"dims": (256, 256, 256), "device_bytes": 4 * 258 ** 3, "code_bytes": 69206016 + 1032}
PLAIN = {"dims": (64, 64, 64), "device_bytes": 4 * 66 ** 3, "code_bytes": 0}


@pytest.mark.parametrize("info,depth,per,held", [(CODED, 8, 1, 258 ** 3), (CODED, 4, 4, 4 * 258 ** 3),
                                                 (PLAIN, 8, 4, 4 * 66 ** 3)])
def test_bytes_of_a_step(info, depth, per, held):
    assert bench.step_bytes(info, depth) == per
    assert bench.step_set(info, depth) == held
    r = bench.roofline_of("k", 1.8e12, bench.step_set(info, depth), CEIL, bench.step_bytes(info, depth))
    assert r["achieved"] == pytest.approx(1800.0 * per)
    assert r["frac"] == pytest.approx(1800.0 * per / 8000.0)
    label = "1MiB" if held <= 4 << 20 else "64MiB"
    assert r["levels"]["ceiling_working_set"] == label
    assert r["levels"]["frac_vs_stream"] == pytest.approx(1800.0 * per / CEIL[label]["stream_gbs"])
