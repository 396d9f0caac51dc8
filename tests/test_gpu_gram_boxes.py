"""The Gram search's tile boxes (up to d = 16) at the sizes where they can go
wrong: tiles of 64 clusters and one more or less, more tiles than one test of 256
takes, clustered inputs whose tiles are mostly skipped, uniform ones whose tiles
are not, and d = 17 without boxes. Tolerances as in the other parity tests."""
import numpy as np
import pytest

import oracle
import synth
from tests import _trees

pytestmark = pytest.mark.gpu

RTOL = {"complete": 0.0, "average": 1e-12, "ward": 0.0, "avgsq": 1e-10}


@pytest.mark.parametrize("link", ["complete", "average", "ward", "avgsq"])
@pytest.mark.parametrize("n,d,kind", [(2, 4, "u"), (63, 9, "b"), (64, 16, "b"), (65, 5, "u"), (129, 17, "b"),
                                      (1000, 9, "u"), (2500, 16, "b"), (17000, 4, "b")])
def test_gram_tile_boxes(link, n, d, kind, monkeypatch):
    import paper_2106_04727_amd as pc

    monkeypatch.setenv("PC_TREE_MAX_DIM", "0")
    monkeypatch.setenv("PC_GRAM_MIN_DIM", "4")  # the Gram search in every round
    x = synth.uniform(n, d, 40 + n) if kind == "u" else synth.blobs(n, d, max(1, n // 100), 0.02, 40 + n)
    if n > 10000 and link in ("complete", "average"):
        # too slow for the oracle: the same rows as the matrix rounds give
        Z = pc.hac(x, link)
        monkeypatch.delenv("PC_TREE_MAX_DIM")
        monkeypatch.delenv("PC_GRAM_MIN_DIM")
        Zo = pc.hac(x, link)
    else:
        Z = pc.hac(x, link)
        Zo, cert = oracle.nnchain(x, link, threads=8)
        assert cert["min_gap"] >= 1e-10 or n < 3, "fixed input no longer certified tie-free"
    _trees.assert_valid(Z, n)
    assert _trees.same_tree(Z, Zo, n, rtol=RTOL[link])
