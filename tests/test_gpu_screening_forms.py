"""The Gram search and its screening tiles in calls that would otherwise start
with the pair matrix or scan rounds: every element type, interval tiles, the
settling pass and its fallback, block boxes of giant pairs. The matrix, the scan
rounds and the box tree are switched off, and the Gram launches are counted, so a
change of the dispatch cannot empty these tests."""
import numpy as np
import pytest

import oracle
import synth
from tests import _trees

pytestmark = pytest.mark.gpu

RTOL = {"complete": 0.0, "ward": 0.0, "average": 1e-12, "avgsq": 1e-10}


@pytest.fixture
def pc(monkeypatch):
    import paper_2106_04727_amd as pc

    monkeypatch.setenv("PC_MATRIX_MAX", "0")
    monkeypatch.setenv("PC_TREE_MAX_DIM", "0")
    return pc


def _run(pc, x, link, precisions=("fp16", "bf16", "fp32")):
    Zo, cert = oracle.nnchain(x, link, threads=8)
    assert cert["min_gap"] >= 1e-10, "fixed input no longer certified tie-free"
    out = []
    for precision in precisions:
        Z, st = pc.hac(x, link, return_stats=True, timing="kernels", precision=precision)
        assert st["kernels"]["ring_search"]["launches"] >= st["rounds"]  # Gram pass 0
        assert st["kernels"]["ring_emit"]["launches"] >= st["rounds"]    # Gram pass 1
        _trees.assert_valid(Z, x.shape[0])
        assert _trees.same_tree(Z, Zo, x.shape[0], rtol=RTOL[link]), precision
        # a candidate per screened chain tail at least: the rest are fallbacks
        assert st["refined"] > 0 and 0 <= st["fp64_fallbacks"] < st["refined"]
        out.append(st)
    return out


@pytest.mark.parametrize("link", ["complete", "average", "ward", "avgsq"])
@pytest.mark.parametrize("n,d,kind,seed", [(3000, 10, "b", 7), (1200, 64, "b", 11), (1000, 128, "s", 12)])
def test_gram_search_forms(pc, link, n, d, kind, seed):
    _run(pc, synth.blobs(n, d, 8, 0.03, seed) if kind == "b" else synth.sphere_blobs(n, d, 25, 0.1, seed), link)


@pytest.mark.parametrize("link", ["complete", "average"])
@pytest.mark.parametrize("d", [40, 64, 128])
def test_interval_tiles(pc, link, d):
    for st in _run(pc, synth.sphere_blobs(1200, d, 12, 0.1, 60 + d), link):
        assert st["kernels"]["block_search"]["visits"] > 0  # point pairs screened


def test_settling_falls_back(pc):
    rng = np.random.default_rng(71)
    g, m, d = 6, 80, 64
    cen = rng.normal(0.0, 3.0, (g, d))
    x = (np.repeat(cen, m, axis=0) + rng.uniform(-1e-4, 1e-4, (g * m, d))).astype(np.float32)
    st, = _run(pc, x, "complete", ("fp16",))
    assert st["kernels"]["pair_tiles"]["launches"] > 0


@pytest.mark.parametrize("d", [5, 8, 12])
def test_giant_pairs(pc, d):
    rng = np.random.default_rng(100 + d)
    x = np.vstack([rng.normal(0.0, 1.0, (2500, d)), rng.normal(0.0, 1.0, (2000, d)) + 6.0]).astype(np.float32)
    st, = _run(pc, x, "complete", ("fp16",))
    assert st["kernels"]["block_search"]["visits"] > 0
