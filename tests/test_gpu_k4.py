"""GPU parity of the 4-clique count (tricc_graph_count_k4) against the
oracle's node iterator: small graphs and closed forms, R-MAT / BA / ER graphs,
a graph built from a CSR, repeat calls, and the out-degree limit. Counts are
integers, compared exactly. Complete graphs K_k reach every kernel: out-degrees
up to 512 (K_513 and below), 513-1,024 (K_514 .. K_1025), the quarter passes
(K_1026 .. K_2049) and the sixteenth passes (K_2050, K_2100); the dense
G(1100, 0.6) case takes the 513-1,024 kernel against the oracle. The pass
kernels also run on sparse rows: hub-and-core graphs whose centres have
out-degrees just above 1,024, inside (1,024, 2,048] and inside
(2,048, 4,096], against stored oracle counts (tests/golden/k4_pass.json)."""
import json
import os
from math import comb

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


def gpu_k4(g):
    out = g.count_k4()
    torch.cuda.synchronize()
    return int(out.cpu().numpy().view(np.uint64)[0])


CASES = [
    ("messy_K9", lambda: F.messy(*F.complete(9), seed=5)),
    ("families", lambda: F.disjoint_union(F.complete(6), F.wheel(3), F.ring_lattice(30, 6), F.windmill(4),
                                          F.grid(5, 5), F.complete_bipartite(4, 5))),
    ("rmat12", lambda: I.rmat(12, 16, seed=51)),
    ("rmat14", lambda: I.rmat(14, 16, seed=52)),
    ("er", lambda: (20000, *I.er(20000, 300000, 53))),
    ("ba", lambda: (20000, *I.ba(20000, 10, 54))),
    ("no_edges", lambda: (9, np.zeros(0, np.int32), np.zeros(0, np.int32))),
]


@pytest.mark.parametrize("name", [c[0] for c in CASES])
def test_against_oracle(name):
    n, s, d = dict(CASES)[name]()
    g = P.Graph(n, dev(s), dev(d))
    ref = oracle.k4(n, s, d, order=1)
    assert gpu_k4(g) == ref
    assert gpu_k4(g) == ref  # repeat calls


@pytest.mark.parametrize("k", [4, 5, 17, 33, 60, 65, 66, 67, 300, 513, 514, 600, 1025, 1026, 1100, 2049, 2050,
                               2100])
def test_complete_graphs(k):
    n, s, d = F.complete(k)
    assert gpu_k4(P.Graph(n, dev(s), dev(d))) == comb(k, 4)


def test_dense_random_graph_against_oracle():
    # G(1100, 0.6): the lowest-ranked nodes keep out-degrees of 512-617,
    # which take the 148 KB bit-row kernel
    n = 1100
    s, d = I.er(n, int(0.6 * n * (n - 1) / 2), 77)
    g = P.Graph(n, dev(s), dev(d))
    assert 512 < g.info["max_outdeg"] <= 1024
    assert gpu_k4(g) == oracle.k4(n, s, d, order=1)


def test_rmat17_and_from_csr():
    n, s, d = I.rmat(17, 16, seed=55)
    ref = oracle.k4(n, s, d, order=1)
    g = P.Graph(n, dev(s), dev(d))
    assert gpu_k4(g) == ref
    a = np.minimum(s, d).astype(np.int64)
    b = np.maximum(s, d).astype(np.int64)
    keep = a != b
    key = np.unique(a[keep] * n + b[keep])
    u, v = key // n, key % n
    rows = np.concatenate([u, v])
    cols = np.concatenate([v, u])
    order = np.lexsort((cols, rows))
    rows, cols = rows[order], cols[order]
    rowptr = np.cumsum(np.concatenate([[0], np.bincount(rows, minlength=n)])).astype(np.int64)
    g2 = P.Graph.from_csr(n, torch.from_numpy(rowptr).to(DEV), dev(cols), assume_simple_sorted_symmetric=True)
    assert gpu_k4(g2) == ref


def test_out_degree_limit_is_enforced():
    n, s, d = F.complete(8194)
    g = P.Graph(n, dev(s), dev(d))
    assert g.info["max_outdeg"] > 8192
    with pytest.raises(N.TriccError) as ei:
        g.count_k4()
    assert ei.value.status == N.TRICC_EOVERFLOW


def _k4_core_cases():
    with open(os.path.join(os.path.dirname(__file__), "golden", "k4_pass.json")) as f:
        return json.load(f)["graphs"]


@pytest.mark.parametrize("case", _k4_core_cases(), ids=lambda c: f"core{c['core']}")
def test_pass_kernels_on_sparse_rows(case):
    """The centres' rows over N+(centre) (the core) are sparse with partial
    last words, so the passes' position filter and hit lists matter."""
    n, s, d = F.k4_core(case["core"], case["centres"], case["avg_deg"], case["seed"])
    assert n == case["n"]
    print(f"[k4] core={case['core']} centres={case['centres']} n={n}", flush=True)
    g = P.Graph(n, dev(s), dev(d))
    mo = g.info["max_outdeg"]
    assert case["core"] <= mo <= case["core"] + case["centres"] - 1 and 1024 < mo <= 8192
    assert gpu_k4(g) == case["k4"]
    assert gpu_k4(g) == case["k4"]


def gpu_k5(g):
    out = g.count_k5()
    torch.cuda.synchronize()
    return int(out.cpu().numpy().view(np.uint64)[0])


K5_CASES = [
    ("messy_K10", lambda: F.messy(*F.complete(10), seed=25)),
    ("families", lambda: F.disjoint_union(F.complete(7), F.wheel(4), F.ring_lattice(40, 8), F.windmill(4),
                                          F.grid(5, 5), F.complete_bipartite(4, 5))),
    ("rmat12", lambda: I.rmat(12, 16, seed=61)),
    ("rmat13", lambda: I.rmat(13, 16, seed=62)),
    ("er", lambda: (20000, *I.er(20000, 300000, 63))),
    ("ba", lambda: (20000, *I.ba(20000, 10, 64))),
    ("dense", lambda: (400, *I.er(400, 40000, 65))),
    ("no_edges", lambda: (9, np.zeros(0, np.int32), np.zeros(0, np.int32))),
]


@pytest.mark.parametrize("name", [c[0] for c in K5_CASES])
def test_k5_against_oracle(name):
    n, s, d = dict(K5_CASES)[name]()
    print(f"[k5] {name} n={n} m_raw={len(s)}", flush=True)
    g = P.Graph(n, dev(s), dev(d))
    ref = oracle.k5(n, s, d, order=1)
    assert gpu_k5(g) == ref
    assert gpu_k5(g) == ref  # repeat calls


@pytest.mark.parametrize("k", [5, 6, 33, 64, 65, 300, 513, 514, 700, 1025])
def test_k5_complete_graphs(k):
    n, s, d = F.complete(k)
    assert gpu_k5(P.Graph(n, dev(s), dev(d))) == comb(k, 5)


def test_k5_out_degree_limit_and_degeneracy():
    n, s, d = F.complete(1026)
    g = P.Graph(n, dev(s), dev(d))
    with pytest.raises(N.TriccError) as ei:
        g.count_k5()
    assert ei.value.status == N.TRICC_EOVERFLOW
    # the same count under the degeneracy order, whose out-degrees stay
    # within the core numbers
    n, s, d = I.rmat(12, 16, seed=66)
    g = P.Graph(n, dev(s), dev(d))
    ref = oracle.k5(n, s, d, order=1)
    assert gpu_k5(g) == ref
    g.orient_degeneracy()
    assert gpu_k5(g) == ref


def _k5_core_cases():
    with open(os.path.join(os.path.dirname(__file__), "golden", "k4_pass.json")) as f:
        return json.load(f).get("k5_graphs", [])


@pytest.mark.parametrize("case", _k5_core_cases(), ids=lambda c: f"core{c['core']}")
def test_k5_larger_kernel_on_sparse_rows(case):
    n, s, d = F.k4_core(case["core"], case["centres"], case["avg_deg"], case["seed"])
    assert n == case["n"]
    g = P.Graph(n, dev(s), dev(d))
    assert 512 < g.info["max_outdeg"] <= 1024
    assert gpu_k5(g) == case["k5"]


def test_k4_complete_graph_above_4096():
    n, s, d = F.complete(4100)
    g = P.Graph(n, dev(s), dev(d))
    assert g.info["max_outdeg"] == 4099
    assert gpu_k4(g) == comb(4100, 4)


@pytest.mark.parametrize("core", [3, 4, 63, 64, 65, 127, 129, 256, 257, 511, 512])
def test_out_degrees_at_the_kernels_edges(core):
    """Centres whose out-degree is `core` (the centres share a random core that
    leaves lift above them in degree), with sparse rows, beside an R-MAT graph
    whose out-degrees take the kernels of smaller rows."""
    rng = np.random.default_rng(core)
    centres = 3
    iu, ju = np.triu_indices(core, 1)
    keep = rng.random(iu.size) < (0.9 if core < 10 else 0.15)
    c = np.repeat(np.arange(core, core + centres), core)
    leaves = centres + 2
    leaf = core + centres + np.arange(core * (core + leaves))
    parts = [(iu[keep], ju[keep]), (c, np.tile(np.arange(core), centres)),
             (np.repeat(np.arange(core), core + leaves), leaf)]
    n1 = int(core + centres + leaf.size)
    n2, s2, d2 = I.rmat(9, 8, seed=core)
    s = np.concatenate([p[0] for p in parts] + [s2.astype(np.int64) + n1])
    d = np.concatenate([p[1] for p in parts] + [d2.astype(np.int64) + n1])
    g = P.Graph(n1 + n2, dev(s), dev(d))
    assert core <= g.info["max_outdeg"] <= max(core, 64)
    assert gpu_k4(g) == oracle.k4(n1 + n2, s, d, order=1)
    assert gpu_k5(g) == oracle.k5(n1 + n2, s, d, order=1)


@pytest.mark.parametrize("k", [2, 70, 300, 600])
def test_place_tables_fall_back_to_buckets(k):
    """Complete graphs whose last four ids agree in their low 24 bits, so that
    they share one slot pair and every table that holds them is rebuilt in the
    bucket layout: in the kernels of out-degrees up to 64, 256, 512 and 1,024."""
    ids = np.concatenate([2 + 27_001 * np.arange(k), 1 + (np.arange(1, 5) << 24)])  # a block takes nodes of close ids
    i, j = np.triu_indices(ids.size, 1)
    g = P.Graph(int(ids[-1]) + 1, dev(ids[i]), dev(ids[j]))
    assert g.info["max_outdeg"] == ids.size - 1
    assert gpu_k4(g) == comb(ids.size, 4)
    assert gpu_k5(g) == comb(ids.size, 5)


@pytest.mark.parametrize("near", [40, 100, 128, 130, 260])
@pytest.mark.parametrize("step", [1, 3])
def test_lists_of_neighbouring_ids(near, step):
    """Rings of nodes joined to the nearest on both sides: lists of consecutive
    ids (or every third), streamed packed and one by one, the longest lists of a
    wavefront's node 64 ids."""
    n = 1500
    n0, s, d = F.ring_lattice(n, near)
    s, d = s.astype(np.int64) * step, d.astype(np.int64) * step
    g = P.Graph(n * step, dev(s), dev(d))
    assert gpu_k4(g) == oracle.k4(n * step, s.astype(np.int32), d.astype(np.int32), order=1)
    assert gpu_k5(g) == oracle.k5(n * step, s.astype(np.int32), d.astype(np.int32), order=1)


@pytest.mark.parametrize("core,density", [(513, 0.02), (600, 0.004), (992, 0.01), (993, 0.001), (1024, 0.02), (1000, 0.0)])
def test_sparse_rows_of_large_out_degrees(core, density):
    """Centres joined to all of a core whose nodes are joined sparsely: rows with
    no bit, one or few, most of their words empty, the last word partly used."""
    rng = np.random.default_rng(core)
    iu, ju = np.triu_indices(core, 1)
    keep = rng.random(iu.size) < density
    centres = 5
    c = np.repeat(np.arange(core, core + centres), core)
    leaves = core + centres + 5  # they lift the core above the centres
    leaf = core + centres + np.arange(core * leaves)
    s = np.concatenate([iu[keep], c, np.repeat(np.arange(core), leaves)])
    d = np.concatenate([ju[keep], np.tile(np.arange(core), centres), leaf])
    n = int(core + centres + leaf.size)
    g = P.Graph(n, dev(s), dev(d))
    assert g.info["max_outdeg"] == core
    assert gpu_k4(g) == oracle.k4(n, s, d, order=1)
    assert gpu_k5(g) == oracle.k5(n, s, d, order=1)
