"""Device bytes that a call reserves: no Gram records for calls that search the box
tree in every round (Ward and avg-2 up to d = 8)."""
import pytest

import paper_2106_04727_amd as pc


@pytest.mark.parametrize("link", ["ward", "avgsq"])
@pytest.mark.parametrize("d", [6, 8])
def test_no_gram_records_with_the_tree(link, d, monkeypatch):
    n = 1_000_000
    monkeypatch.delenv("PC_TREE_MAX_DIM", raising=False)
    tree = pc.workspace_bytes(n, d, link)
    monkeypatch.setenv("PC_TREE_MAX_DIM", "0")  # the Gram search instead
    gram = pc.workspace_bytes(n, d, link)
    # 4n candidates of 64 bytes and more, 16 FP16 coordinates and a norm record per point
    assert gram - tree >= 4 * n * 64 + n * (16 * 2 + 16)


def test_the_gram_search_keeps_its_records(monkeypatch):
    monkeypatch.delenv("PC_TREE_MAX_DIM", raising=False)
    n = 100_000
    for link, d in (("ward", 9), ("avgsq", 128), ("complete", 4), ("average", 64)):
        assert pc.workspace_bytes(n, d, link) > 4 * n * 64 + n * 4 * d
