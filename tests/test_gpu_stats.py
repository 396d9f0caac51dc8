"""Counters of calls that keep a pair matrix or scan all clusters."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("link", ["complete", "average", "ward", "avgsq"])
def test_unscreened_pairs_are_no_fallbacks(link):
    """Calls that only keep a matrix or scan: every pair gets its exact value, and
    none of them because a tile could not rule it out."""
    import paper_2106_04727_amd as pc

    _, st = pc.hac(synth.blobs(1500, 10, 20, 0.03, 5), link, return_stats=True, timing="kernels")
    assert st["kernels"]["ring_search"]["launches"] == 0
    assert st["refined"] > 0 and st["fp64_fallbacks"] == 0


@pytest.mark.parametrize("link,loads", [("ward", 4), ("avgsq", 4), ("complete", 4), ("average", 8)])
def test_box_tree_visits_are_loads(link, loads, monkeypatch):
    """Two points: a leaf of two clusters and a box on each of the two levels,
    loaded once by a wavefront that serves both terminals (complete linkage
    searches its first round as Ward), or by a wavefront for each (average)."""
    import paper_2106_04727_amd as pc

    monkeypatch.setenv("PC_TREE_MAX_DIM", "8")
    monkeypatch.setenv("PC_FULL_SCAN_MAX", "0")
    _, st = pc.hac(synth.uniform(2, 2, 3), link, return_stats=True)
    assert st["rounds"] == 1
    assert st["kernels"]["ring_search"]["visits"] == loads
