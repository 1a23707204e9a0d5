"""Rules of the library's host side, from a CPU build of its headers: which storage order an
autotuner keeps of those it timed."""

import ctypes as C
import importlib.util
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    spec = importlib.util.spec_from_file_location("_rules_build", os.path.join(
        os.path.dirname(HERE), "paper_2503_22588_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    lib = str(tmp_path_factory.mktemp("rules") / "rules.so")
    cmd = [build.hipcc(), *build.COMMON, "--offload-host-only", "-shared", "-o", lib,
           os.path.join(HERE, "host_rules_check.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return C.CDLL(lib)


@pytest.mark.parametrize("ms,current,margin,kept", [
    ([8.10, 8.10, 8.09, 8.11], 1, 0.02, 1),            # equal walks: noise moves nothing
    ([8.10, 8.10, 8.09, 8.11], 3, 0.02, 3),
    ([8.10, 8.10, 8.09, 8.11], 1, 0.0, 2),             # without a margin the fastest
    ([16.0, 9.0, 11.0, 10.0], 0, 0.02, 1),             # orders that matter
    ([16.0, 9.0, 11.0, 10.0], 1, 0.02, 1),
    ([8.0, 9.0, 8.1, 8.9], 1, 0.02, 0),
    ([8.0, 8.0, 8.0, 8.0], 2, 0.0, 2),
])
def test_order_kept(rules, ms, current, margin, kept):
    a = np.array(ms, np.float32)
    assert rules.pick_layout(a.ctypes.data_as(C.c_void_p), 4, current, C.c_float(margin)) == kept
