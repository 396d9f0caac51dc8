"""Sums of the pair matrix under average linkage when it is entered with
clusters: the same bits in every run, and the values of the other searches.
Clusters across windows of 64 positions and across units (two windows, or more
where few clusters hold many points), giant clusters beside single points, both
kernels (d <= 16 and above). Heights within 1e-12 of the search without a matrix
(a mean of N FP64 terms in another order)."""
import numpy as np
import pytest

import oracle
import synth
from tests import _trees

pytestmark = pytest.mark.gpu


def _points(kind, n, d):
    if kind == "blobs":
        return synth.blobs(n, d, max(1, n // 600), 0.02, 5 + n + d)
    rng = np.random.default_rng(n + d)  # "giants": two dense groups and far single points
    x = rng.normal(0.0, 1.0, (n, d))
    x[: n // 3] += 40.0
    x[-n // 20 :] *= 300.0
    return x[rng.permutation(n)].astype(np.float32)


@pytest.mark.parametrize("kind,n,d,cap", [
    ("blobs", 129, 2, 40), ("blobs", 1025, 3, 300), ("blobs", 60_000, 2, None), ("blobs", 20_000, 2, 60),
    ("blobs", 9_001, 10, 1_000), ("blobs", 9_000, 20, 3_000), ("blobs", 20_000, 20, 60), ("giants", 20_011, 2, 2_000),
    ("giants", 12_000, 3, 100), ("giants", 9_000, 17, 500)])
def test_average_sums(kind, n, d, cap, monkeypatch):
    import paper_2106_04727_amd as pc

    x = _points(kind, n, d)
    monkeypatch.setenv("PC_MATRIX_MAX", "0")
    Z0 = pc.hac(x, "average")
    if cap is None:
        monkeypatch.delenv("PC_MATRIX_MAX")
    else:
        monkeypatch.setenv("PC_MATRIX_MAX", str(cap))
    Z = pc.hac(x, "average")
    _trees.assert_valid(Z, n)
    assert _trees.same_tree(Z, Z0, n, rtol=1e-12)
    for _ in range(3):
        assert np.array_equal(Z, pc.hac(x, "average"))


def test_average_height_error():
    """Heights over many point pairs against long double means. Two roundings are
    left at the end, of the sum and of the quotient, each at most one unit of 2^-53
    relative and evenly spread (rms at most 1 / sqrt(3)); the errors of the single
    distances (a few units) average out below 0.2 units over 256 pairs or more.
    Together an rms of at most 0.85 units."""
    import paper_2106_04727_amd as pc

    n, d = 7151, 64
    x = synth.blobs(n, d, 40, 0.03, 3)
    Z = pc.hac(x, "average")
    members = {i: np.array([i]) for i in range(n)}
    err = []
    for r, (a, b, h, size) in enumerate(Z):
        A, B = members.pop(int(a)), members.pop(int(b))
        members[n + r] = np.concatenate([A, B])
        pairs = A.size * B.size
        if not 256 <= pairs < 65536 or (pairs < 2048 and r % 4):
            continue
        q = np.zeros((A.size, B.size), np.longdouble)
        for k in range(d):
            u = x[A, k, None].astype(np.float64) - x[None, B, k].astype(np.float64)
            q += u.astype(np.longdouble) ** 2
        exact = np.sqrt(q).sum() / pairs
        err.append(float((np.longdouble(h) - exact) / exact) * 2.0 ** 53)
    assert len(err) > 50
    assert np.sqrt(np.mean(np.square(err))) <= 0.85


@pytest.mark.parametrize("n,d", [(130, 3), (130, 20), (700, 200)])
@pytest.mark.parametrize("scale", [3.4e38, 1e-36, 1e-43])
def test_average_at_the_ends_of_the_range(n, d, scale):
    """Coordinates next to the largest floats, and so small that they lose bits:
    squared distances from 2^-290 to 2^266."""
    import paper_2106_04727_amd as pc

    x = (synth.uniform(n, d, 17).astype(np.float64) * 2.0 - 1.0) * scale
    x = x.astype(np.float32)
    assert np.isfinite(x).all()
    Z = pc.hac(x, "average")
    _trees.assert_valid(Z, n)
    Zo, cert = oracle.nnchain(x, "average", threads=8)
    assert cert["min_gap"] >= 1e-10, "fixed input no longer certified tie-free"
    assert _trees.same_tree(Z, Zo, n, rtol=1e-12)
