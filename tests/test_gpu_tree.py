"""The box-tree searches (Ward and avg-2 up to d = 8, complete and average up
to d = 3) at the sizes where it can go wrong:
leaves of 64 clusters and one more or less, one and two levels above them,
groups of four terminals with a remainder, every width of the coordinate loops,
ties, outliers, flat inputs and overflowing records. Ward and complete heights
are the oracle's bit for bit, average heights within 1e-12 (a mean of N FP64
terms in another order), avg-2 heights within 1e-10 (spreads by an equivalent
merge rule)."""
import numpy as np
import pytest

import oracle
import synth
from tests import _trees

pytestmark = pytest.mark.gpu

RTOL = {"ward": 0.0, "avgsq": 1e-10, "complete": 0.0, "average": 1e-12}


@pytest.fixture
def pc(monkeypatch):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2106_04727_amd as pc

    pc.load_library()
    monkeypatch.setenv("PC_TREE_MAX_DIM", "8")
    monkeypatch.setenv("PC_FULL_SCAN_MAX", "0")  # the tree in every round
    return pc


@pytest.mark.parametrize("link", ["ward", "avgsq"])
@pytest.mark.parametrize("n,d", [(2, 1), (5, 2), (63, 2), (64, 3), (65, 5), (130, 8), (700, 7), (4096, 2), (4097, 1),
                                 (4100, 6), (5003, 4)])
def test_tree_rounds(pc, link, n, d):
    x = synth.blobs(n, d, max(1, n // 80), 0.03, 700 + n + d)
    Zo, cert = oracle.nnchain(x, link, threads=8)
    Z, st = pc.hac(x, link, return_stats=True)
    assert st["kernels"]["ring_search"]["visits"] > 0
    _trees.assert_valid(Z, n)
    if cert["min_gap"] >= 1e-10 or n < 3:
        assert _trees.same_tree(Z, Zo, n, rtol=RTOL[link])
    else:
        _trees.assert_valid_hac(x, Z, link, rtol=1e-9)


@pytest.mark.parametrize("link", ["ward", "avgsq"])
def test_tree_ties_outliers_and_flat_inputs(pc, link):
    g = np.stack(np.meshgrid(np.arange(13.0), np.arange(9.0)), -1).reshape(-1, 2).astype(np.float32)
    _trees.assert_valid_hac(g, pc.hac(g, link), link, rtol=1e-9)  # a lattice: equal keys everywhere
    x = synth.uniform(150, 3, 8)
    x = np.concatenate([x, x])  # every point twice
    Z = pc.hac(x, link)
    _trees.assert_valid_hac(x, Z, link, rtol=1e-9)
    assert np.all(Z[:150, 2] == 0.0)
    x = synth.uniform(900, 3, 9)
    x[::90] *= 1e4  # far outliers stretch the curve's cells and the boxes
    x[:, 1] = 0.5   # one axis without extent
    Zo, _ = oracle.nnchain(x, link, threads=8)
    assert _trees.same_tree(pc.hac(x, link), Zo, 900, rtol=RTOL[link])


@pytest.mark.parametrize("link", ["complete", "average"])
@pytest.mark.parametrize("n,d", [(2, 1), (5, 2), (63, 2), (64, 3), (65, 3), (700, 1), (4096, 2), (4097, 3), (4500, 2)])
@pytest.mark.parametrize("slots", [0, 64])
def test_tree_pair_rounds(pc, link, n, d, slots):
    x = synth.blobs(n, d, max(1, n // 80), 0.03, 700 + n + d)
    Zo, cert = oracle.nnchain(x, link, threads=8)
    Z, st = pc.hac(x, link, return_stats=True, cache_slots=slots)
    assert st["kernels"]["ring_search"]["visits"] > 0
    _trees.assert_valid(Z, n)
    if cert["min_gap"] >= 1e-10 or n < 3:
        assert _trees.same_tree(Z, Zo, n, rtol=RTOL[link])
    else:
        _trees.assert_valid_hac(x, Z, link, rtol=1e-9)


@pytest.mark.parametrize("link", ["complete", "average"])
def test_tree_pair_ties_and_overflow(pc, link, monkeypatch):
    g = np.stack(np.meshgrid(np.arange(11.0), np.arange(9.0)), -1).reshape(-1, 2).astype(np.float32)
    _trees.assert_valid_hac(g, pc.hac(g, link), link, rtol=1e-9)
    x = synth.uniform(150, 3, 8)
    Z = pc.hac(np.concatenate([x, x]), link)
    assert np.all(Z[:150, 2] == 0.0) and Z[150, 2] > 0.0
    x = synth.blobs(3000, 2, 10, 0.03, 33)
    Zo, _ = oracle.nnchain(x, link, threads=8)
    for cap in ("16", "400"):  # a record too small for the walk: the round runs again on the grid
        monkeypatch.setenv("PC_TEST_CAND_CAP", cap)
        assert _trees.same_tree(pc.hac(x, link), Zo, 3000, rtol=RTOL[link])


@pytest.mark.parametrize("kind", ["u", "b"])
def test_complete_plane_grid_or_tree(kind):
    """Rounds above and below 60,000 active clusters, on evenly spread points
    (ring searches down to there) and on mixtures (box tree from the third round):
    the same rows, exactly, as the accelerated oracle's."""
    import paper_2106_04727_amd as pc

    n = 100_000
    x = synth.uniform(n, 2, 71) if kind == "u" else synth.blobs(n, 2, 50, 0.01, 72)
    Z = pc.hac(x, "complete")
    Zo, cert = oracle.nnchain(x, "complete", threads=8, accel=True)
    assert cert["min_gap"] >= 1e-10, "fixed input no longer certified tie-free"
    _trees.assert_valid(Z, n)
    assert _trees.same_tree(Z, Zo, n, rtol=0.0)
