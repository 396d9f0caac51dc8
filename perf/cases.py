"""Measured cases: the clustering calls a user of this library makes.

Each case is one call (or one burst of server requests) through the package's
public entry points:

* ``device``   ``hac_device`` on a float32 tensor on the GPU (rows stay there);
* ``host``     ``hac`` on a host array (copy in, rows out as a linkage matrix);
* ``noalloc``  ``Context.hac_noalloc`` into the caller's row buffer;
* ``server``   a burst of requests submitted to a ``Server`` from host arrays.

The point laws are the ones the library is used and tested on: isotropic
Gaussian mixtures in the unit cube, uniform points, unit vectors around random
centres, and the UniformFill / GaussianDisc laws of the ParChain paper
(Sec. 6). Outputs are the whole dendrogram: children, heights and sizes of
every row.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2106_04727_amd as pc

LINKAGES = ("complete", "average", "ward", "avgsq")


def _case(name, entry, linkage, law, n, d, k=0, sigma=0.0, precision="fp16"):
    return {"name": name, "entry": entry, "linkage": linkage, "law": law, "n": n, "d": d,
            "k": k, "sigma": sigma, "precision": precision}


def listed():
    return [
        # the smallest request of the serving law: latency of one call
        _case("n256_d2_ward", "device", "ward", "blobs", 256, 2, 5, 0.03),
        # the parity set's size, from a host array to a linkage matrix: the
        # scipy-style call of an interactive user
        _case("host_2k_d2_complete", "host", "complete", "uniform", 2_000, 2),
        # a mid-size request in the serving law's highest dimension, odd size
        _case("n7151_d64_average", "device", "average", "blobs", 7_151, 64, 40, 0.03),
        # a caller that must not allocate (its own row buffer), 3-D, odd size
        _case("noalloc_20011_d3_average", "noalloc", "average", "blobs", 20_011, 3, 50, 0.02),
        # many small requests of uneven shape at once
        {"name": "server_burst_24", "entry": "server", "count": 24, "mix": 41, "n_hi": 20_000, "slots": 4},
        # the headline pair: 1M points in the plane, both linkages
        _case("blob50_1m_d2_ward", "device", "ward", "blobs", 1_000_000, 2, 50, 0.01),
        _case("blob50_1m_d2_complete", "device", "complete", "blobs", 1_000_000, 2, 50, 0.01),
        # the largest point count
        _case("blob50_10m_d2_ward", "device", "ward", "blobs", 10_000_000, 2, 50, 0.01),
        # the paper's planar set under mean-distance linkage
        _case("disc_500k_d2_average", "device", "average", "gaussian_disc", 500_000, 2),
        # the paper's 5-D set under mean squared distance
        _case("fill_1m_d5_avgsq", "device", "avgsq", "uniform_fill", 1_000_000, 5),
        # ten-dimensional mixture under mean-distance linkage, odd size
        _case("blob100_250007_d10_average", "device", "average", "blobs", 250_007, 10, 100, 0.02),
        # embedding-like unit vectors, BF16 screening tiles
        _case("sphere_50k_d128_complete_bf16", "device", "complete", "sphere", 50_000, 128, 1000, 0.1, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["small", "small", "plane", "plane", "average2", "mid", "deep", "server"])
    k, sigma = rng.randint(5, 100), rng.uniform(0.01, 0.05)
    if kind == "small":
        entry = rng.choice(["device", "device", "host", "noalloc"])
        n = _log_int(rng, 256, 20_000)
        return _case(None, entry, rng.choice(LINKAGES), rng.choice(["blobs", "uniform"]), n,
                     rng.choice([2, 3, 5, 10, 64]), k, sigma)
    if kind == "plane":
        law = rng.choice(["blobs", "uniform_fill", "gaussian_disc"])
        n = _log_int(rng, 20_000, 10_000_000)
        return _case(None, "device", rng.choice(["ward", "complete", "avgsq"]), law, n, 2, k, sigma)
    if kind == "average2":
        n = _log_int(rng, 20_000, 500_000)
        law = rng.choice(["blobs", "uniform_fill", "gaussian_disc"])
        return _case(None, "device", "average", law, n, rng.choice([2, 3]) if n < 300_000 else 2, k, sigma)
    if kind == "mid":
        link = rng.choice(["ward", "avgsq", "average"])
        n = _log_int(rng, 20_000, 1_000_000 if link != "average" else 200_000)
        d = rng.choice([3, 4, 5]) if link != "average" else rng.choice([5, 10])
        return _case(None, "device", link, "blobs" if link == "average" else "uniform_fill", n, d, k, sigma)
    if kind == "deep":
        n = _log_int(rng, 5_000, 30_000)
        return _case(None, "device", rng.choice(LINKAGES), "sphere", n, rng.choice([64, 100, 128]),
                     rng.choice([50, 300, 1000]), 0.1, rng.choice(["fp16", "bf16", "fp32"]))
    return {"name": None, "entry": "server", "count": rng.randint(8, 24), "mix": rng.randint(1, 10_000),
            "n_hi": _log_int(rng, 2_000, 20_000), "slots": rng.choice([2, 4, 8])}


# ------------------------------------------------------------------ inputs --

def _points(law, n, d, k, sigma, seed, device):
    """n float32 points, drawn in float64 on `device` and rounded once."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    kw = {"generator": g, "device": device, "dtype": torch.float64}
    if law == "uniform":
        x = torch.rand((n, d), **kw)
    elif law == "blobs":
        centres = torch.rand((k, d), **kw)
        lab = torch.randint(0, k, (n,), generator=g, device=device)
        x = centres[lab] + sigma * torch.randn((n, d), **kw)
    elif law == "sphere":
        c = torch.randn((k, d), **kw)
        c = c / c.norm(dim=1, keepdim=True)
        lab = torch.randint(0, k, (n,), generator=g, device=device)
        x = c[lab] + sigma * torch.randn((n, d), **kw)
        x = x / x.norm(dim=1, keepdim=True)
    elif law == "uniform_fill":
        x = torch.rand((n, d), **kw) * math.sqrt(n)
    elif law == "gaussian_disc":
        side = 5.0 * math.sqrt(n)
        means = torch.rand((5, d), **kw) * side
        ng = int(round(0.9 * n))
        lab = torch.arange(ng, device=device) % 5
        x = torch.cat([means[lab] + torch.randn((ng, d), **kw) * (math.sqrt(n) / 6.0),
                       torch.rand((n - ng, d), **kw) * side])
        x = x[torch.randperm(n, generator=g, device=device)]
    else:
        raise ValueError(law)
    return x.to(torch.float32).contiguous()


def _requests(case, seed):
    """The burst's requests: sizes log-uniform, shapes of the serving law.

    The mix of shapes is the case's, the points are the seed's.
    """
    rng = np.random.default_rng(case["mix"])
    reqs = []
    for i in range(case["count"]):
        n = int(np.exp(rng.uniform(np.log(256), np.log(case["n_hi"]))))
        d = int(rng.choice([2, 3, 10, 64]))
        link = str(rng.choice(["complete", "average", "ward"]))
        k, sigma = int(rng.integers(5, 101)), float(rng.uniform(0.01, 0.05))
        reqs.append((link, n, d, k, sigma, 1000 * seed + i))
    return reqs


def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _server_inputs(case, seed):
    return [(link, _points("blobs", n, d, k, sigma, s, "cpu").numpy())
            for link, n, d, k, sigma, s in _requests(case, seed)]


def _inputs(case, seed):
    device = "cpu" if case["entry"] == "host" else _device()
    return _points(case["law"], case["n"], case["d"], case["k"], case["sigma"], seed, device)


def prepare(case, seed):
    if case["entry"] == "server":
        return {"case": case, "server": pc.Server(slots=case["slots"]), "requests": _server_inputs(case, seed)}
    x = _inputs(case, seed)
    state = {"case": case, "x": x.numpy() if case["entry"] == "host" else x}
    if case["entry"] == "noalloc":
        state["ctx"] = pc.Context(_device().index)
        state["rows"] = torch.empty((case["n"] - 1, 4), dtype=torch.int64, device=x.device)
    return state


# -------------------------------------------------------------------- pass --

def _split_rows(rows):
    return {"a": rows[:, 0], "b": rows[:, 1], "height": rows[:, 2].view(torch.float64), "size": rows[:, 3]}


def _from_host(rows):
    """The host entries' layout of the exact rows."""
    return {"merges": np.stack([rows["a"], rows["b"], rows["size"]], axis=1), "height": rows["height"]}


def _split_Z(Z):
    return {"merges": Z[:, [0, 1, 3]].astype(np.int64), "height": Z[:, 2]}


def run(state):
    case = state["case"]
    if case["entry"] == "server":
        srv = state["server"]
        tickets = [srv.submit(x, link) for link, x in state["requests"]]
        return [_split_Z(srv.result(t)[0]) for t in tickets]
    x = state["x"]
    if case["entry"] == "host":
        return _split_Z(pc.hac(x, case["linkage"], precision=case["precision"]))
    if case["entry"] == "noalloc":
        rows = state["rows"]
        state["ctx"].hac_noalloc(x.data_ptr(), case["n"], case["d"], case["linkage"], rows.data_ptr(),
                                 stream=torch.cuda.current_stream().cuda_stream, precision=case["precision"])
        return _split_rows(rows)
    rows, _ = pc.hac_device(x, case["linkage"], precision=case["precision"])
    return _split_rows(rows)


# -------------------------------------------------------------------- work --

def _work(linkage, n, d):
    nbytes = 4 * n * d + 32 * (n - 1)
    if linkage == "average":
        # every point pair's distance is part of exactly one merge's mean
        flops = (3 * d + 1) * n * (n - 1) // 2
    else:
        # one nearest neighbour per point and one distance per merge, 3 d each
        flops = 3 * d * (2 * n - 1)
    return nbytes, flops


def work(case):
    if case["entry"] == "server":
        parts = [_work(link, n, d) for link, n, d, _, _, _ in _requests(case, 0)]
    else:
        parts = [_work(case["linkage"], case["n"], case["d"])]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ------------------------------------------------------------------- exact --

_EXACT_MAX_N = 8_000


def _pair_sq(x):
    """All squared distances in float64, coordinates summed in order."""
    dev = _device() if torch.cuda.is_available() else torch.device("cpu")
    xt = torch.as_tensor(x).to(dev, torch.float64)
    n, d = xt.shape
    out = torch.zeros((n, n), dtype=torch.float64, device=dev)
    for j in range(d):
        t = xt[:, j, None] - xt[None, :, j]
        out += t * t
    return out.cpu().numpy()


def _chain(M, update):
    """Nearest-neighbour chain over the key matrix M (overwritten).

    ``update(row_a, row_b, i, j, size)`` gives the merged cluster's keys. Returns
    the merges as (slot kept, slot dropped) pairs in merge order.
    """
    n = M.shape[0]
    np.fill_diagonal(M, np.inf)
    size = np.ones(n)
    alive = np.ones(n, bool)
    chain, merges, low = [], [], 0
    while len(merges) < n - 1:
        if not chain:
            while not alive[low]:
                low += 1
            chain.append(low)
        i = chain[-1]
        j = int(np.argmin(M[i]))
        if len(chain) > 1 and M[i, chain[-2]] <= M[i, j]:
            j = chain[-2]
            del chain[-2:]
            a, b = min(i, j), max(i, j)
            row = update(M[a], M[b], a, b, size)
            row[a] = np.inf
            row[~alive] = np.inf
            row[b] = np.inf
            M[a] = row
            M[:, a] = row
            M[b] = np.inf
            M[:, b] = np.inf
            size[a] += size[b]
            alive[b] = False
            merges.append((a, b))
        else:
            chain.append(j)
    return merges


def _exact_rows(linkage, x):
    x = np.asarray(x, np.float64)
    n = x.shape[0]
    D = _pair_sq(x)
    if linkage in ("average", "complete"):
        D = np.sqrt(D)
    if linkage == "complete":
        def update(ra, rb, a, b, size):
            return np.maximum(ra, rb)
    elif linkage == "ward":
        def update(ra, rb, a, b, size):
            sa, sb = size[a], size[b]
            return ((sa + size) * ra + (sb + size) * rb - size * ra[b]) / (sa + sb + size)
    else:
        def update(ra, rb, a, b, size):
            sa, sb = size[a], size[b]
            return (sa * ra + sb * rb) / (sa + sb)
    merges = _chain(D.copy(), update)
    # heights from their definitions over the two children's points
    members = {i: np.array([i]) for i in range(n)}
    h = np.empty(n - 1)
    m = np.empty(n - 1, np.int64)
    for r, (a, b) in enumerate(merges):
        A, B = members[a], members.pop(b)
        if linkage == "ward":
            gap = x[A].mean(axis=0) - x[B].mean(axis=0)
            h[r] = math.sqrt(2.0 * A.size * B.size / (A.size + B.size) * float((gap * gap).sum()))
        else:
            block = D[A[:, None], B[None, :]]
            h[r] = block.max() if linkage == "complete" else float(block.mean(dtype=np.longdouble))
        members[a] = np.concatenate([A, B])
        m[r] = members[a].size
    # row order: largest height of the subtree, size, lowest point index
    eff = np.empty(n - 1)
    top = {}
    for r, (a, b) in enumerate(merges):
        eff[r] = max(h[r], top.get(a, 0.0), top.get(b, 0.0))
        top[a] = eff[r]
    low = np.array([a for a, _ in merges])  # the kept slot is the lowest point index
    order = np.lexsort((low, m, eff))
    node = {i: i for i in range(n)}
    kids = []
    for r, (a, b) in enumerate(merges):
        kids.append((node[a], node[b]))
        node[a] = n + r
    new = np.empty(n - 1, np.int64)
    new[order] = np.arange(n - 1)

    def label(v):
        return v if v < n else n + int(new[v - n])

    ab = np.array([sorted((label(p), label(q))) for p, q in kids], np.int64)
    return {"a": ab[order, 0], "b": ab[order, 1], "height": h[order], "size": m[order]}


def exact(case, seed):
    if case["entry"] == "server":
        return [_from_host(_exact_rows(link, x)) if x.shape[0] <= 2_000 else {"merges": None, "height": None}
                for link, x in _server_inputs(case, seed)]
    if case["n"] > _EXACT_MAX_N:
        return None
    rows = _exact_rows(case["linkage"], _inputs(case, seed).cpu().numpy())
    return _from_host(rows) if case["entry"] == "host" else rows
