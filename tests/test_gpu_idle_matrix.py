"""A pair matrix kept from an earlier call gives way to a later call's buffers
when the device has no other memory for them."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_idle_matrix_gives_way():
    import torch
    from paper_2106_04727_amd import parchain

    ctx = parchain.Context(0)
    n, d = 200_000, 8
    a = torch.from_numpy(synth.blobs(16_000, 20, 40, 0.02, 1)).cuda()
    b = torch.from_numpy(synth.blobs(n, d, 50, 0.02, 2)).cuda()
    ref = parchain.hac_device(b, "ward")[0]
    out = torch.empty_like(ref)
    need = parchain.workspace_bytes(n, d, "ward")
    parchain.hac_device(a, "complete", ctx=ctx)  # keeps a matrix of 4 GB
    torch.cuda.empty_cache()
    # leave less than the second call's workspace
    fill = []
    for _ in range(8):
        left = torch.cuda.mem_get_info()[0]
        if left < need // 2:
            break
        fill.append(torch.empty(left - need // 4, dtype=torch.uint8, device="cuda"))
    try:
        ctx.hac(b.data_ptr(), n, d, "ward", out.data_ptr(), points_on_device=True, out_on_device=True,
                stream=torch.cuda.current_stream().cuda_stream)
    finally:
        fill.clear()
        torch.cuda.empty_cache()
        ctx.close()
    assert left < need // 2
    assert torch.equal(out, ref)
