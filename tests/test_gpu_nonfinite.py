"""Non-finite coordinates in a tensor on the device: refused by every linkage
and entry point, whatever the values do to the kernels that are queued before
the host reads the check, and without a trace in the context's next call. Sizes:
rounds in one block alone (50), matrix and scan rounds before them (700), and
more points than those take (17,000)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

NAN, INF = np.float32(np.nan), np.float32(np.inf)


def _spoil(x, how):
    x = x.copy()
    if how == "one nan":
        x[len(x) // 2, -1] = NAN
    elif how == "all nan":
        x[:] = NAN
    elif how == "inf in the first point":
        x[0, 0] = INF
    elif how == "-inf in the last point":
        x[-1, -1] = -INF
    elif how == "a column of inf":
        x[:, 0] = INF
    elif how == "all but two points inf":
        x[2:] = INF
    return x


@pytest.mark.parametrize("link", ["complete", "average", "ward", "avgsq"])
@pytest.mark.parametrize("n,d", [(2, 1), (50, 2), (700, 2), (700, 20), (17_000, 2)])
def test_nonfinite_on_the_device(link, n, d):
    import torch
    from paper_2106_04727_amd import PCError, parchain

    x = synth.blobs(n, d, max(1, n // 60), 0.03, 61)
    xd = torch.from_numpy(x).cuda()
    ctx = parchain.Context(0)
    ref, _ = parchain.hac_device(xd, link, ctx=ctx)
    out = torch.empty((n - 1, 4), dtype=torch.int64, device="cuda")
    for how in ("one nan", "all nan", "inf in the first point", "-inf in the last point", "a column of inf",
                "all but two points inf"):
        bad = torch.from_numpy(_spoil(x, how)).cuda()
        if bool(torch.isfinite(bad).all()):
            continue  # (two points: nothing to spoil)
        with pytest.raises(PCError) as e:
            parchain.hac_device(bad, link, ctx=ctx)
        assert e.value.status == -2, how
        out.fill_(-7)
        with pytest.raises(PCError) as e:
            ctx.hac_noalloc(bad.data_ptr(), n, d, link, out.data_ptr(),
                            stream=torch.cuda.current_stream().cuda_stream)
        assert e.value.status == -2, how
        assert bool((out == -7).all())
        rows, _ = parchain.hac_device(xd, link, ctx=ctx)
        ids = [0, 1, 3]
        assert torch.equal(rows[:, ids], ref[:, ids]), how
        assert torch.allclose(rows[:, 2].view(torch.float64), ref[:, 2].view(torch.float64), rtol=1e-12, atol=0.0)
    ctx.close()
