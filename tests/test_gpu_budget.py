"""A budget of exactly pc_hac_workspace_bytes holds a call whose records need not
grow, from host and device points, on every search."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("link", ["complete", "average", "ward", "avgsq"])
@pytest.mark.parametrize("n,d", [(8, 3), (3000, 2), (40_000, 2), (20_000, 6), (9_000, 12), (2_000, 64)])
def test_the_stated_workspace_is_enough(link, n, d):
    import numpy as np
    import torch
    from paper_2106_04727_amd import parchain

    x = synth.blobs(n, d, max(1, n // 100), 0.02, 70 + n + d)
    xd = torch.from_numpy(x).cuda()
    ref = parchain.rows_to_Z(parchain.hac_device(xd, link)[0])
    ctx = parchain.Context(0, hbm_budget_bytes=parchain.workspace_bytes(n, d, link))
    Z = parchain.rows_to_Z(parchain.hac_device(xd, link, ctx=ctx)[0])
    out = np.zeros((n - 1, 4), np.int64)
    ctx.hac(x.ctypes.data, n, d, link, out.ctypes.data, points_on_device=False, out_on_device=False)
    ctx.close()
    for got in (Z, parchain.rows_to_Z(out)):
        assert np.array_equal(got[:, [0, 1, 3]], ref[:, [0, 1, 3]])
        assert np.allclose(got[:, 2], ref[:, 2], rtol=1e-12 if link == "average" else 0.0, atol=0.0)
