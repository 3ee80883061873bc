"""GPU parity of the edge-existence tests (tricc_graph_has_edges) against the
oracle's search in the sorted edge set: every pair of small graphs (and ids
outside [0, n)), mixed true and random queries on R-MAT and on the paper's
smallest edge-test configuration (G(n=1M, m=10M), one random query per
edge), graphs built from edge lists and from a CSR, and the call's error
paths. Results are uint8 codes, compared exactly."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1606_07550_amd as P
from paper_1606_07550_amd import _native as N
from paper_1606_07550_amd import inputs as I
from paper_1606_07550_amd.inputs import fixtures as F

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def gpu_has(g, qu, qv):
    out = g.has_edges(dev(qu), dev(qv))
    torch.cuda.synchronize()
    return out.cpu().numpy()


def all_pairs(n):
    qu, qv = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    bad_u = np.array([-1, n, 0, n + 5, -7, 2**31 - 1])
    bad_v = np.array([0, 0, n, 1, -1, 0])
    return (np.concatenate([qu.ravel(), bad_u]).astype(np.int32),
            np.concatenate([qv.ravel(), bad_v]).astype(np.int32))


def mixed_queries(n, s, d, k, seed):
    """k queries: half input pairs in a random direction, half random pairs."""
    rng = np.random.default_rng(seed)
    h = k // 2
    e = rng.integers(0, s.size, h)
    flip = rng.integers(0, 2, h).astype(bool)
    qu = np.concatenate([np.where(flip, d[e], s[e]), rng.integers(0, n, k - h)]).astype(np.int32)
    qv = np.concatenate([np.where(flip, s[e], d[e]), rng.integers(0, n, k - h)]).astype(np.int32)
    return qu, qv


SMALL = [
    ("messy_K8", lambda: F.messy(*F.complete(8), seed=3)),
    ("wheel", lambda: F.wheel(17)),
    ("star", lambda: F.star(25)),
    ("windmill", lambda: F.windmill(6)),
    ("rmat8", lambda: I.rmat(8, 8, seed=4)),
    ("er", lambda: (60, *I.er(60, 400, 5))),
    ("loops_only", lambda: (5, np.array([0, 1, 2], np.int32), np.array([0, 1, 2], np.int32))),
    ("no_edges", lambda: (7, np.zeros(0, np.int32), np.zeros(0, np.int32))),
]


@pytest.mark.parametrize("name", [c[0] for c in SMALL])
def test_every_pair_of_small_graphs(name):
    n, s, d = dict(SMALL)[name]()
    qu, qv = all_pairs(n)
    g = P.Graph(n, dev(s), dev(d))
    np.testing.assert_array_equal(gpu_has(g, qu, qv), oracle.has_edges(n, s, d, qu, qv))


def test_rmat16_true_random_and_hub_queries():
    n, s, d = I.rmat(16, 16, seed=31)
    g = P.Graph(n, dev(s), dev(d))
    qu, qv = mixed_queries(n, s, d, 1 << 20, 32)
    # the largest hub against every id, both ways round
    hub = int(np.argmax(g.arrays()["deg"].cpu().numpy()))
    ids = np.arange(n, dtype=np.int32)
    qu = np.concatenate([qu, np.full(n, hub, np.int32), ids])
    qv = np.concatenate([qv, ids, np.full(n, hub, np.int32)])
    got = gpu_has(g, qu, qv)
    ref = oracle.has_edges(n, s, d, qu, qv)
    np.testing.assert_array_equal(got, ref)
    first = slice(0, 1 << 19)
    assert got[first][qu[first] != qv[first]].all()  # every input pair but a loop is an edge


def test_graph_from_csr_and_edge_list_agree():
    n, s, d = I.rmat(12, 16, seed=33)
    a = np.minimum(s, d).astype(np.int64)
    b = np.maximum(s, d).astype(np.int64)
    keep = a != b
    key = np.unique(a[keep] * n + b[keep])
    u, v = key // n, key % n
    rows = np.concatenate([u, v])
    cols = np.concatenate([v, u])
    order = np.lexsort((cols, rows))
    rows, cols = rows[order], cols[order]
    rowptr = np.zeros(n + 1, np.int64)
    np.add.at(rowptr, rows + 1, 1)
    rowptr = np.cumsum(rowptr)
    g = P.Graph.from_csr(n, torch.from_numpy(rowptr).to(DEV), dev(cols), assume_simple_sorted_symmetric=True)
    qu, qv = mixed_queries(n, s, d, 200000, 34)
    np.testing.assert_array_equal(gpu_has(g, qu, qv), oracle.has_edges(n, s, d, qu, qv))


def test_paper_config_er_1m_10m():
    """G(n=1M, m=10M) with one random query per edge (Section 6.2's smallest
    edge-test graph), plus every input pair."""
    n, m = 1_000_000, 10_000_000
    s, d = I.er(n, m, 35)
    g = P.Graph(n, dev(s), dev(d))
    rng = np.random.default_rng(36)
    qu = np.concatenate([rng.integers(0, n, m), s]).astype(np.int32)
    qv = np.concatenate([rng.integers(0, n, m), d]).astype(np.int32)
    got = gpu_has(g, qu, qv)
    np.testing.assert_array_equal(got, oracle.has_edges(n, s, d, qu, qv))
    assert got[m:].all()


def test_empty_queries_and_errors():
    n, s, d = F.complete(6)
    g = P.Graph(n, dev(s), dev(d))
    e = torch.empty(0, dtype=torch.int32, device=DEV)
    assert g.has_edges(e, e).numel() == 0
    L = N.lib()
    assert L.tricc_graph_has_edges(None, 1, None, None, None, None) == N.TRICC_EINVAL
    assert L.tricc_graph_has_edges(g._h, -1, None, None, None, None) == N.TRICC_EINVAL
    assert L.tricc_graph_has_edges(g._h, 4, None, None, None, None) == N.TRICC_EINVAL
    assert L.tricc_graph_has_edges(g._h, 0, None, None, None, None) == N.TRICC_OK
    with pytest.raises(ValueError):
        g.has_edges(dev([0, 1]), torch.zeros(2, dtype=torch.int64, device=DEV))
    # results do not depend on the stream or on a count running before them
    qu, qv = all_pairs(n)
    o = g.count()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        out = g.has_edges(dev(qu), dev(qv), stream=side)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), oracle.has_edges(n, s, d, qu, qv))
    assert int(o["total"].cpu().numpy().view(np.uint64)[0]) == 20


@pytest.mark.parametrize("more", [0, 600_000, 2_800_000], ids=["halving", "blocks_of_8", "blocks_of_16"])
@pytest.mark.parametrize("spread", ["even", "low", "high", "two_ends"])
def test_rows_at_the_edges_of_blocks(spread, more):
    """Rows of 1 to 140 ids at every offset against blocks of 8 and 16, their ids
    spread evenly or clustered, tested with every id that any row holds and with
    the ids beside them; the other ends have longer rows. More pairs, among ids
    that no test names, take the graph to each of the row searches."""
    n, pool = 100_000, 150
    ids = {"even": np.linspace(400, n - 2, pool).astype(np.int64), "low": 400 + 2 * np.arange(pool),
           "high": n - 2 * pool + 2 * np.arange(pool),
           "two_ends": np.concatenate([400 + np.arange(pool // 2) * 3, n - pool + np.arange(pool // 2) * 2])}[spread]
    rng = np.random.default_rng(len(spread))
    lens = np.concatenate([np.arange(1, 71), [95, 96, 97, 127, 128, 129, 140]])
    s = [np.full(k, u) for u, k in enumerate(lens)]
    d = [rng.choice(ids, k, replace=False) for k in lens]
    fill = 100 + np.arange(160)  # they lift the degrees of the ids above the rows' lengths
    keys = np.unique(np.concatenate([ids, ids - 1, np.minimum(ids + 1, n - 1), [0, n - 1]]))
    others = np.setdiff1d(np.arange(1000, n), keys)
    s = np.concatenate(s + [np.repeat(fill, pool), rng.choice(others, more)])
    d = np.concatenate(d + [np.tile(ids, fill.size), rng.choice(others, more)])
    g = P.Graph(n, dev(s), dev(d))
    m = g.info["m"]
    assert (m < 5 * n, 8 * m > 20 << 20) == {0: (True, False), 600_000: (False, False), 2_800_000: (False, True)}[more]
    qu, qv = (a.ravel() for a in np.meshgrid(np.arange(lens.size), keys, indexing="ij"))
    want = np.isin(qu * n + qv, np.concatenate([s * n + d, d * n + s])).astype(np.uint8)
    np.testing.assert_array_equal(gpu_has(g, qu, qv), want)
    np.testing.assert_array_equal(gpu_has(g, qv, qu), want)


@pytest.mark.parametrize("hub", [0, 64, 65])
def test_short_rows_of_a_large_graph(hub):
    """A ring of a million nodes, each joined to the next two: rows of 4 ids,
    searched by halving, and by blocks once one row is longer than 64."""
    n = 1_000_003
    i = np.arange(n)
    s, d = np.concatenate([i, i]), np.concatenate([(i + 1) % n, (i + 2) % n])
    far = 500_000 + 7 * np.arange(max(hub - 4, 0))
    s, d = np.concatenate([s, np.full(far.size, 10)]), np.concatenate([d, far])
    g = P.Graph(n, dev(s), dev(d))
    assert g.info["max_deg"] == (hub or 4) and 2 * g.info["m"] <= 5 * n and 8 * g.info["m"] > 12 << 20
    u = np.repeat(np.concatenate([i[:40], i[-40:], far[:5], [10]]), 9)
    v = (u + np.tile(np.arange(-4, 5), u.size // 9)) % n
    u, v = np.concatenate([u, np.full(far.size, 10), np.full(far.size, 10)]), np.concatenate([v, far, far + 1])
    gap = np.minimum((u - v) % n, (v - u) % n)
    want = ((gap == 1) | (gap == 2) | ((u == 10) & np.isin(v, far)) | ((v == 10) & np.isin(u, far))).astype(np.uint8)
    np.testing.assert_array_equal(gpu_has(g, u, v), want)
    np.testing.assert_array_equal(gpu_has(g, v, u), want)


@pytest.mark.parametrize("top", [1, 50])
def test_rows_where_degrees_lie_unevenly(top):
    """The first block is guessed from where the degrees lie: all of them at the
    low or at the high ids, rows there and away from there, every id tested."""
    n, m = 60_000, 400_000
    rng = np.random.default_rng(top)
    s = rng.integers(0, n, m)
    d = (rng.random(m) ** 6 * n).astype(np.int64)
    if top == 50:
        s, d = n - 1 - s, n - 1 - d
    g = P.Graph(n, dev(s), dev(d))
    keep = s != d
    key = np.unique(np.concatenate([s[keep] * n + d[keep], d[keep] * n + s[keep]]))
    ids = np.concatenate([rng.integers(0, n, 40), d[:40], [0, n - 1]])
    u, v = (a.ravel() for a in np.meshgrid(ids, np.arange(0, n, 7), indexing="ij"))
    u, v = np.concatenate([u, key // n]), np.concatenate([v, key % n])
    want = np.isin(u * n + v, key).astype(np.uint8)
    np.testing.assert_array_equal(gpu_has(g, u, v), want)


@pytest.mark.parametrize("more", [0, 600_000, 2_800_000], ids=["halving", "blocks_of_8", "blocks_of_16"])
@pytest.mark.parametrize("q", [3 << 16, (3 << 16) + 1, 500_001])
def test_few_and_many_queries(q, more):
    """Few tests go by halving, more by the row search that the graph's size
    asks for: rows of 1 to 140 ids at every offset against blocks of 8 and 16,
    their ids spread evenly, in one clump or at both ends, tested with every id
    that a row holds and the ids beside it, and with ids outside [0, n)."""
    n, pool = 100_000, 150
    rng = np.random.default_rng(q)
    ids = [np.linspace(400, n - 2, pool).astype(np.int64), 50_000 + 2 * np.arange(pool),
           np.concatenate([600 + np.arange(pool // 2) * 3, n - 400 + np.arange(pool // 2) * 2])]
    lens = np.tile(np.concatenate([np.arange(1, 71), [95, 96, 97, 127, 128, 129, 140]]), 3)
    s = [np.full(k, u) for u, k in enumerate(lens)]
    d = [rng.choice(ids[u * 3 // lens.size], k, replace=False) for u, k in enumerate(lens)]
    keys = np.unique(np.concatenate([x + o for x in ids for o in (-1, 0, 1)] + [[0, n - 1]]))
    fill = 240 + np.arange(160)  # they lift the degrees of the rows' ids above the rows' lengths
    others = np.setdiff1d(np.arange(1000, n), keys)
    s = np.concatenate(s + [np.repeat(fill, 3 * pool), rng.choice(others, more)])
    d = np.concatenate(d + [np.tile(np.concatenate(ids), fill.size), rng.choice(others, more)])
    g = P.Graph(n, dev(s), dev(d))
    m = g.info["m"]
    assert (m < 5 * n, 8 * m > 20 << 20) == {0: (True, False), 600_000: (False, False), 2_800_000: (False, True)}[more]
    qu, qv = (a.ravel() for a in np.meshgrid(np.arange(lens.size), keys, indexing="ij"))
    qu, qv = np.resize(qu, q), np.resize(qv, q)
    want = np.isin(qu * n + qv, np.concatenate([s * n + d, d * n + s])).astype(np.uint8)
    bad = np.arange(0, q, 997)
    qv[bad], want[bad] = np.where(bad % 2, n, -1), 0xFF
    np.testing.assert_array_equal(gpu_has(g, qu, qv), want)
    np.testing.assert_array_equal(gpu_has(g, qv, qu), want)


@pytest.mark.parametrize("name", ["K41", "K30_30"])
def test_few_queries_of_dense_graphs(name):
    """Dense graphs go by blocks however few the tests are."""
    n, s, d = F.complete(41) if name == "K41" else F.complete_bipartite(30, 30)
    g = P.Graph(n, dev(s), dev(d))
    assert 8 * g.info["m"] >= n * n and g.info["m"] >= 5 * n
    qu, qv = all_pairs(n)
    np.testing.assert_array_equal(gpu_has(g, qu, qv), oracle.has_edges(n, s, d, qu, qv))
