"""The memory a map says it takes, words and codes, against what the device has less of."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,coded", [((64, 64, 64), False), ((100, 100, 100), True), ((256, 256, 256), True),
                                         ((320, 320, 320), True), ((254, 254, 200), True), ((2000, 1500, 1), True), ((5, 1500, 1000), False),
                                         ((6, 1500, 1000), True),
                                         ((1022, 1, 4000), True)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_memory_of_words_and_codes(shape, coded):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_22588_amd as nbt
    print(f"[gpu] memory of a {shape} map", flush=True)
    nx, ny, nz = shape
    P = torch.full((nz, ny, nx), 0.5, device="cuda")
    ctx = nbt.Context(0)
    ctx.set_map_layout(nbt.LAYOUT_LINEAR)
    nbt.Map(ctx, P[:1].contiguous(), 0.1, (0.0, 0.0, 0.0)).close()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    m = nbt.Map(ctx, P, 0.1, (0.0, 0.0, 0.0))
    took = before - torch.cuda.mem_get_info()[0]
    i = m.info()
    assert i["device_bytes"] == 4 * (nx + 2) * (ny + 2) * (nz + 2)
    field = lambda n: max(8, 1 << (n + 1).bit_length())  # noqa: E731
    want = field(nx) * field(ny) * -(-(nz + 2) // 8) * 8
    assert i["code_bytes"] == (want + 258 * 4 if coded else 0)
    assert i["code_bytes"] <= 2.7 * i["device_bytes"] + 2048
    if min(shape) >= 100:
        assert i["code_bytes"] <= 1.07 * i["device_bytes"] + 2048
    assert abs(took - i["device_bytes"] - i["code_bytes"]) <= 3 * (2 << 20)      # whole 2 MiB pieces of each allocation
    ctx.close()
