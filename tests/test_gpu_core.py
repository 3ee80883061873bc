"""GPU parity of the core numbers (tricc_graph_core) against the oracle's
Batagelj-Zaversnik bucket algorithm: small families and closed forms with
several stop levels, R-MAT / BA / ER graphs, a graph built from a CSR, repeat
calls, the empty graph and the call's error paths. Core numbers are
integers, compared exactly."""
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


def gpu_core(g, k_stop=-1):
    c, mx = g.core(k_stop)
    torch.cuda.synchronize()
    return c.cpu().numpy(), mx


CASES = [
    ("messy_K9", lambda: F.messy(*F.complete(9), seed=5)),
    ("families", lambda: F.disjoint_union(F.wheel(12), F.windmill(5), F.star(6), F.complete(5), F.grid(4, 6),
                                          F.complete_bipartite(3, 7), F.ring_lattice(30, 4), F.path(9))),
    ("rmat10", lambda: I.rmat(10, 8, seed=6)),
    ("er", lambda: (3000, *I.er(3000, 20000, 7))),
    ("ba", lambda: (5000, *I.ba(5000, 6, 8))),
    ("isolated", lambda: (6, np.array([1, 2], np.int32), np.array([2, 1], np.int32))),
    ("no_edges", lambda: (9, np.zeros(0, np.int32), np.zeros(0, np.int32))),
]


@pytest.mark.parametrize("name", [c[0] for c in CASES])
def test_small_graphs_every_stop_level(name):
    n, s, d = dict(CASES)[name]()
    g = P.Graph(n, dev(s), dev(d))
    for k in (-1, 0, 1, 2, 3, 5):
        got, mx = gpu_core(g, k)
        ref = oracle.core(n, s, d, k)
        np.testing.assert_array_equal(got, ref, err_msg=f"k_stop {k}")
        assert mx == (int(ref.max()) if n else 0)


def test_rmat16_and_repeat_calls():
    n, s, d = I.rmat(16, 16, seed=41)
    g = P.Graph(n, dev(s), dev(d))
    ref = oracle.core(n, s, d)
    a, mx = gpu_core(g)
    np.testing.assert_array_equal(a, ref)
    assert mx == ref.max()
    b, _ = gpu_core(g)
    np.testing.assert_array_equal(a, b)
    three, _ = gpu_core(g, 3)
    np.testing.assert_array_equal(three, np.minimum(ref, 3))


def test_rmat20_full_decomposition():
    n, s, d = I.rmat(20, 16, seed=20)
    g = P.Graph(n, dev(s), dev(d))
    got, mx = gpu_core(g)
    ref = oracle.core(n, s, d)
    np.testing.assert_array_equal(got, ref)
    assert mx == ref.max()


def test_graph_from_csr():
    n, s, d = I.rmat(12, 16, seed=43)
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
    g = P.Graph.from_csr(n, torch.from_numpy(rowptr).to(DEV), dev(cols), assume_simple_sorted_symmetric=True)
    got, _ = gpu_core(g)
    np.testing.assert_array_equal(got, oracle.core(n, s, d))


def test_empty_graph_and_errors():
    g0 = P.Graph(0, dev([]), dev([]))
    c, mx = g0.core()
    assert c.numel() == 0 and mx == 0
    n, s, d = F.complete(7)
    g = P.Graph(n, dev(s), dev(d))
    L = N.lib()
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    need = ctypes.c_size_t()
    assert L.tricc_core_workspace_size(n, ctypes.byref(need)) == N.TRICC_OK
    ws = torch.empty(need.value, dtype=torch.uint8, device=DEV)
    mx = ctypes.c_int32()
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.tricc_graph_core(None, -1, None, None, 0, None, sp) == N.TRICC_EINVAL
    assert L.tricc_graph_core(g._h, -1, ctypes.c_void_p(out.data_ptr()), None, 0, None, sp) == N.TRICC_EINVAL
    assert L.tricc_graph_core(g._h, -1, ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(ws.data_ptr()),
                              need.value - 1, None, sp) == N.TRICC_ENOMEM
    assert L.tricc_graph_core(g._h, -1, ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(ws.data_ptr()),
                              need.value, ctypes.byref(mx), sp) == N.TRICC_OK
    assert mx.value == 6 and bool((out == 6).all().item())


def rounds(n, s, d):
    """Core numbers and removal rounds by peeling level by level: all nodes of
    current degree at most k together, a level's rounds numbered from a
    multiple of four."""
    keep = s != d
    key = np.unique(np.concatenate([s[keep].astype(np.int64) * n + d[keep], d[keep].astype(np.int64) * n + s[keep]]))
    u, w = key // n, key % n
    off = np.searchsorted(u, np.arange(n + 1))
    cur = np.diff(off)
    core, order, k, r = np.full(n, -1), np.zeros(n, np.int64), 0, 0
    while (core < 0).any():
        k = max(k, cur[core < 0].min())
        F, first = np.flatnonzero((core < 0) & (cur <= k)), r
        while F.size:
            core[F], order[F] = k, r
            r += 1
            at = np.repeat(off[F] - np.concatenate([[0], np.cumsum(np.diff(off)[F])[:-1]]), np.diff(off)[F])
            nb = w[at + np.arange(at.size)]
            cur -= np.bincount(nb, minlength=n)
            F = np.unique(nb[(core[nb] < 0) & (cur[nb] <= k)])
        r = first + (r - first + 3) // 4 * 4
        k += 1
    return core, order


def hubs_with_leaves(hubs, leaves, tail):
    """`hubs` stars whose centres fall due in the second round, when their rows
    are long, together with the second nodes of as many paths of `tail` nodes."""
    n1 = hubs * (leaves + 1)
    h = np.repeat(np.arange(hubs), leaves)
    n2 = hubs * tail
    p = n1 + np.arange(n2).reshape(hubs, tail)
    s = np.concatenate([h, p[:, :-1].ravel()])
    d = np.concatenate([hubs + np.arange(hubs * leaves), p[:, 1:].ravel()])
    return n1 + n2, s.astype(np.int32), d.astype(np.int32)


# frontiers below, at and above the bounds of the peel's ways: 512 nodes, the
# launch's blocks (1,024), eight nodes to each of its wavefronts (32,768)
FRONTIERS = {
    **{f"bipartite_{a}_{b}": (lambda a=a, b=b: F.complete_bipartite(a, b))
       for a, b in [(100, 511), (100, 512), (100, 513), (100, 1024), (65, 1025), (64, 20_000), (100, 32_768),
                    (100, 32_769), (100, 40_000), (3, 40_000)]},
    **{f"hubs_{h}_{k}": (lambda h=h, k=k: hubs_with_leaves(h, k, 6))
       for h, k in [(1, 3000), (300, 70), (900, 64), (900, 65), (5000, 66), (33_000, 66)]},
    "grid": lambda: F.grid(400, 300),
    "ring_lattice": lambda: F.ring_lattice(30_000, 20),
}


@pytest.mark.parametrize("name", list(FRONTIERS))
def test_frontiers_of_every_size(name):
    n, s, d = FRONTIERS[name]()
    s, d = np.asarray(s, np.int32), np.asarray(d, np.int32)
    g = P.Graph(n, dev(s), dev(d))
    ref = oracle.core(n, s, d)
    for k in (-1, 2, 3, 34):
        got, mx = gpu_core(g, k)
        np.testing.assert_array_equal(got, ref if k < 0 else np.minimum(ref, k), err_msg=f"k_stop {k}")
        assert mx == int(ref.max() if k < 0 else min(ref.max(), k))
    core, order = rounds(n, s, d)
    np.testing.assert_array_equal(core, ref)
    got = g.degeneracy()
    np.testing.assert_array_equal(got[1].cpu().numpy(), ref)
    np.testing.assert_array_equal(got[0].cpu().numpy(), order)
