"""Rules of the library's host side, from a CPU build of its headers: which storage order an
autotuner keeps of those it timed, and the threads of the planner's cost terms."""

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


@pytest.mark.parametrize("nb,np_", [(1, 1), (1, 10), (2, 10), (10, 500), (1000, 1000)])
def test_cost_threads(rules, nb, np_):
    """A launch has less than 2^32 threads, up to the most states a call accepts (below 2^31)."""
    rules.cost_threads.restype = C.c_ulonglong
    for steps in [*range(1, 67), 100, 1000]:
        for states in (steps, 10 ** 6 // steps * steps, (2 ** 31 - 1) // steps * steps, 2 ** 30 // steps * steps):
            threads = rules.cost_threads(C.c_uint32(states), C.c_uint32(steps), C.c_uint32(nb), C.c_uint32(np_), 256)
            assert states <= threads < 2 ** 32, (states, steps)
