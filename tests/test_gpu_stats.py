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
