"""A pair matrix kept from an earlier call gives way to a later call's buffers
when the device has no other memory for them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_idle_matrix_gives_way():
    import torch
    from paper_2106_04727_amd import parchain

    ctx = parchain.Context(0)
    a = torch.from_numpy(synth.blobs(16_000, 20, 40, 0.02, 1)).cuda()
    b = torch.from_numpy(synth.blobs(200_000, 8, 50, 0.02, 2)).cuda()
    ref = parchain.hac_device(b, "ward")[0]
    need = parchain.workspace_bytes(200_000, 8, "ward")
    parchain.hac_device(a, "complete", ctx=ctx)  # keeps a matrix of 4 GB
    torch.cuda.empty_cache()
    # leave less than the second call's workspace
    fill = []
    for _ in range(8):
        left = torch.cuda.mem_get_info()[0]
        if left < need // 5:
            break
        fill.append(torch.empty(left - need // 8, dtype=torch.uint8, device="cuda"))
    try:
        rows, _ = parchain.hac_device(b, "ward", ctx=ctx)
        same = torch.equal(rows, ref)
    finally:
        fill.clear()
        torch.cuda.empty_cache()
        ctx.close()
    assert left < need // 5 and same
