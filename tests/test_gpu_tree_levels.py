"""The box tree with four levels of 64 children below the first nodes tested: more
than 64^4 active clusters. The rows of the centroid grid, exactly."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("link", ["ward", "avgsq"])
def test_tree_of_four_levels(link, monkeypatch):
    import torch
    from paper_2106_04727_amd import parchain

    n = 64 ** 4 + 12_345
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    x = torch.rand((n, 2), generator=g, device="cuda", dtype=torch.float64).to(torch.float32)
    ctx = parchain.Context(0)
    monkeypatch.delenv("PC_TREE_MAX_DIM", raising=False)
    tree, _ = parchain.hac_device(x, link, ctx=ctx)
    monkeypatch.setenv("PC_TREE_MAX_DIM", "0")
    grid, _ = parchain.hac_device(x, link, ctx=ctx)
    same = torch.equal(tree, grid)
    ctx.close()
    del x, tree, grid
    torch.cuda.empty_cache()
    assert same
