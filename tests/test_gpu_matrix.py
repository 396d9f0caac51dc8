"""Pair-matrix rounds (complete and average linkage) and scan rounds (Ward and
avg-2) at the sizes where their kernels can go wrong: windows of 64 points and
one point more or less, rounds entered with single points or with clusters that
lie across windows, every width of the coordinate loops, ties, and inputs whose
matrix does not fit.

Tolerances are those of the other parity tests: complete
and Ward heights are the oracle's bit for bit, average heights within 1e-12 (a
mean of N FP64 terms in another order differs by at most (N - 1) 2^-53
relative), avg-2 heights within 1e-10 (spreads by an equivalent merge rule)."""
import numpy as np
import pytest

import oracle
import synth
from tests import _trees

pytestmark = pytest.mark.gpu

LINKS = ["complete", "average", "ward", "avgsq"]
RTOL = {"complete": 0.0, "average": 1e-12, "ward": 0.0, "avgsq": 1e-10}


@pytest.fixture(scope="module")
def pc():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2106_04727_amd as pc

    pc.load_library()
    return pc


@pytest.mark.parametrize("link", LINKS)
@pytest.mark.parametrize("n,d", [(2, 1), (3, 2), (63, 2), (64, 3), (65, 5), (129, 10), (700, 2), (1500, 6), (1100, 8),
                                 (2300, 9), (130, 16), (900, 17), (257, 64), (400, 200)])
def test_matrix_rounds(pc, link, n, d, monkeypatch):
    """Entered with the points, later with clusters, and not at all."""
    x = synth.blobs(n, d, max(1, n // 60), 0.03, 900 + n + d)
    Zo, cert = oracle.nnchain(x, link, threads=8)
    assert cert["min_gap"] >= 1e-10 or n < 3, "fixed input no longer certified tie-free"
    for cap in (None, n // 3, n // 12, 0):
        if cap is None:
            monkeypatch.delenv("PC_MATRIX_MAX", raising=False)
        else:
            monkeypatch.setenv("PC_MATRIX_MAX", str(cap))
        Z = pc.hac(x, link)
        _trees.assert_valid(Z, n)
        assert _trees.same_tree(Z, Zo, n, rtol=RTOL[link]), (link, n, d, cap)


@pytest.mark.parametrize("link", LINKS)
@pytest.mark.parametrize("cap", [None, 60])
def test_matrix_ties(pc, link, cap, monkeypatch):
    """Lattice points and points given twice: equal keys everywhere."""
    if cap is not None:
        monkeypatch.setenv("PC_MATRIX_MAX", str(cap))
    g = np.stack(np.meshgrid(np.arange(9.0), np.arange(9.0)), -1).reshape(-1, 2).astype(np.float32)
    _trees.assert_valid_hac(g, pc.hac(g, link), link, rtol=1e-9)
    x = synth.uniform(150, 3, 7)
    x = np.concatenate([x, x])
    Z = pc.hac(x, link)
    _trees.assert_valid_hac(x, Z, link, rtol=1e-9)
    assert np.all(Z[:150, 2] == 0.0) and Z[150, 2] > 0.0
    Z = pc.hac(np.ones((70, 20), np.float32), link)
    assert np.all(Z[:, 2] == 0.0)


@pytest.mark.parametrize("link", ["complete", "average"])
def test_matrix_without_room(pc, link):
    """A budget below the matrix: the call goes on without it; with a little
    more room the matrix is entered once fewer clusters are active."""
    import torch
    from paper_2106_04727_amd import parchain

    n = 6000
    x = torch.from_numpy(synth.blobs(n, 2, 30, 0.02, 77)).cuda()
    ref, _ = parchain.hac_device(x, link)
    base = pc.workspace_bytes(n, 2, link)
    for room in (base + (64 << 20), base + (96 << 20), base + (300 << 20)):
        ctx = parchain.Context(0, hbm_budget_bytes=room)
        rows, _ = parchain.hac_device(x, link, ctx=ctx)
        Za, Zb = parchain.rows_to_Z(ref), parchain.rows_to_Z(rows)
        assert np.array_equal(Za[:, [0, 1, 3]], Zb[:, [0, 1, 3]])
        assert np.allclose(Za[:, 2], Zb[:, 2], rtol=RTOL[link], atol=0.0)
        ctx.close()


@pytest.mark.parametrize("n", [16385, 16386])
def test_row_order_by_rank_and_by_sort(pc, n):
    """16384 rows are ordered by counting, one row more by the radix sorts."""
    x = synth.blobs(n, 2, 300, 0.01, 31)
    Zo, _ = oracle.nnchain(x, "ward", threads=8)
    assert np.array_equal(pc.hac(x, "ward"), oracle.canonical(Zo, n))
