"""Performance cases: the work a user has this library do, through its public
entry points, from the smallest graph to the largest benchmark graph.

Kinds
  count      edge list -> per-node triangles and clustering coefficients, the
             whole path (``count(n, src, dst)``: build + count)
  recount    the count alone, on a graph that the program keeps resident
  csr        the whole path from a sorted, symmetric CSR the caller holds
  batch      many small graphs, packed: build, plan and one run
  batch_run  a planned batch, run again
  serve      induced-subgraph queries (node lists in host memory) against a
             server over a resident graph, to their results
  edges      edge-existence tests against a resident graph
  core       core numbers (k_stop < 0: full decomposition) of a resident graph
  cliques    4- or 5-clique count of a resident graph

Graphs: "rmat" is the package's R-MAT generator, its 2**scale ids folded onto
n and relabelled (heavy tail, duplicates, self loops, both directions of an
edge); "er" draws both ends uniformly (duplicates and self loops occur too).
"""
import math

import numpy as np
import torch

import paper_1606_07550_amd as P

DEV = "cuda"


def listed():
    return [
        # one small graph, alone: an ego network or a molecule; latency and launches
        {"name": "count_er_1k", "kind": "count", "family": "er", "n": 1000, "m": 5003},
        # the quick-start size of the smoke test
        {"name": "count_er_10k", "kind": "count", "family": "er", "n": 10_000, "m": 100_000},
        # an ordinary social graph with ragged sizes
        {"name": "count_rmat_240k", "kind": "count", "family": "rmat", "n": 240_007, "m": 3_900_001},
        # the benchmark's graph: R-MAT scale 24, edge factor 16
        {"name": "count_rmat_16m", "kind": "count", "family": "rmat", "n": 1 << 24, "m": 1 << 28},
        # the golden test's mid size, counted again while it stays resident
        {"name": "recount_rmat_1m", "kind": "recount", "family": "rmat", "n": 1 << 20, "m": 1 << 24},
        # the same graph handed over as the sorted neighbour vectors of a graph store
        {"name": "csr_rmat_1m", "kind": "csr", "family": "rmat", "n": 1 << 20, "m": 1 << 24},
        # a mini-batch of mixed graphs from a data loader, used once
        {"name": "batch_200", "kind": "batch", "graphs": 200, "nmin": 64, "nmax": 65_536},
        # the batched benchmark's 4,096 graphs, planned once and run again
        {"name": "batch_run_4096", "kind": "batch_run", "graphs": 4096, "nmin": 64, "nmax": 65_536},
        # neighbourhood queries of 16 .. 100,000 nodes against a resident graph
        {"name": "serve_100", "kind": "serve", "family": "rmat", "n": 1 << 20, "m": 1 << 24, "queries": 100,
         "kmin": 16, "kmax": 100_000},
        # a block of random edge tests
        {"name": "edges_4m", "kind": "edges", "family": "rmat", "n": 1 << 22, "m": 1 << 26, "queries": 4_000_003},
        # full core decomposition
        {"name": "core_rmat_1m", "kind": "core", "family": "rmat", "n": 1 << 20, "m": 1 << 24, "k_stop": -1},
        # motif count one size above the triangle
        {"name": "k4_rmat_240k", "kind": "cliques", "family": "rmat", "n": 240_007, "m": 3_900_001, "k": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count", "count", "count", "recount", "csr", "batch", "batch_run", "serve", "edges", "core",
                       "cliques"])
    c = {"kind": kind}
    if kind in ("batch", "batch_run"):
        c["graphs"] = _log_int(rng, 2, 2000)
        c["nmin"] = _log_int(rng, 20, 300)
        c["nmax"] = _log_int(rng, 2000, 65_536)
        return c
    top = {"count": 1 << 23, "recount": 1 << 22, "csr": 1 << 22, "serve": 1 << 20, "edges": 1 << 22, "core": 1 << 20,
           "cliques": 1 << 18}[kind]
    c["family"] = rng.choice(["rmat", "er"])
    c["n"] = _log_int(rng, 500, top)
    c["m"] = int(c["n"] * rng.uniform(3.0, 16.0))
    if kind == "serve":
        c["queries"] = _log_int(rng, 1, 200)
        c["kmin"] = 16
        c["kmax"] = max(17, min(100_000, c["n"] // 4))
    elif kind == "edges":
        c["queries"] = _log_int(rng, 1000, 20_000_000)
    elif kind == "core":
        c["k_stop"] = rng.choice([-1, -1, 3])
    elif kind == "cliques":
        c["k"] = rng.choice([4, 4, 5])
    return c


# ---------------------------------------------------------------------------
# inputs, on the GPU, from the seed alone

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _pairs(case, seed):
    n, m, g = case["n"], case["m"], _gen(seed)
    if case["family"] == "er":
        return (torch.randint(n, (m,), generator=g, device=DEV, dtype=torch.int32),
                torch.randint(n, (m,), generator=g, device=DEV, dtype=torch.int32))
    scale = max(1, (n - 1).bit_length())
    perm = torch.randperm(1 << scale, generator=g, device=DEV, dtype=torch.int32)
    if n != 1 << scale:
        perm.remainder_(n)
    return P.generators.rmat(scale, m=m, seed=seed, perm=perm, device=DEV)


def _simple_csr(n, src, dst):
    """Sorted symmetric rows without duplicates and loops: (rowptr, col)."""
    s, d = src.long(), dst.long()
    key = torch.minimum(s, d) * n + torch.maximum(s, d)
    key = torch.unique(key[s != d])
    a, b = key // n, key % n
    both = torch.sort(torch.cat([key, b * n + a]))[0]
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(both // n, minlength=n), 0)
    return rowptr, (both % n).int()


def _batch_pairs(case, seed):
    """Half uniform graphs, half with preferential attachment (a node's
    targets drawn with the limiting degree profile of the Barabasi-Albert
    process: earlier ids in proportion to 1 / sqrt(id)). The sizes belong to
    the case; the seed draws the edges."""
    r = np.random.default_rng([case["graphs"], case["nmin"], case["nmax"]])
    G = case["graphs"]
    n = np.rint(np.exp(r.uniform(math.log(case["nmin"]), math.log(case["nmax"]), G))).astype(np.int64)
    pref = r.random(G) < 0.5
    k = np.where(pref, r.integers(2, 17, G), 0)
    m = np.where(pref, n * k, np.rint(n * r.uniform(2.0, 16.0, G)).astype(np.int64))
    node_off, edge_off = np.zeros(G + 1, np.int64), np.zeros(G + 1, np.int64)
    np.cumsum(n, out=node_off[1:])
    np.cumsum(m, out=edge_off[1:])
    g, M = _gen(seed), int(edge_off[-1])
    m_d = torch.from_numpy(m).to(DEV)

    def spread(a):
        return torch.repeat_interleave(torch.from_numpy(np.ascontiguousarray(a)).to(DEV), m_d, output_size=M)

    nn, kk = spread(n.astype(np.int32)), spread(k.astype(np.int32))
    e = torch.arange(M, device=DEV, dtype=torch.int32) - spread(edge_off[:-1].astype(np.int32))
    x = torch.rand(M, generator=g, device=DEV)
    y = torch.rand(M, generator=g, device=DEV)
    src = torch.where(kk > 0, e // torch.clamp(kk, min=1), torch.minimum((x * nn).int(), nn - 1))
    dst = torch.where(kk > 0, (y * y * src).int(), torch.minimum((y * nn).int(), nn - 1))
    return node_off, edge_off, src.int(), dst.int()


def _balls(case, seed, src, dst):
    """BFS balls of log-uniform size around random nodes that have a
    neighbour, the last level cut at the size: host int32 arrays."""
    n = case["n"]
    off, adj = _simple_csr(n, src, dst)
    deg = off[1:] - off[:-1]
    r = np.random.default_rng(seed)
    has = torch.nonzero(deg > 0).flatten()
    seeds = has[torch.from_numpy(r.integers(0, has.numel(), case["queries"])).to(DEV)]
    seen = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    out = []
    for q in range(case["queries"]):
        k = int(round(math.exp(r.uniform(math.log(case["kmin"]), math.log(case["kmax"])))))
        level = seeds[q:q + 1]
        seen[level] = q
        ball, size = [level], 1
        while size < k and level.numel():
            level = level[:k]
            dl = deg[level]
            first = torch.repeat_interleave(off[level] - (torch.cumsum(dl, 0) - dl), dl)
            nxt = torch.unique(adj[first + torch.arange(first.numel(), device=DEV)]).long()
            level = nxt[seen[nxt] != q][:k - size]
            seen[level] = q
            ball.append(level)
            size += level.numel()
        out.append(torch.cat(ball).int().cpu().numpy())
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "batch_run"):
        node_off, edge_off, src, dst = _batch_pairs(case, seed)
        if kind == "batch":
            return {"case": case, "args": (node_off, edge_off, src, dst)}
        b = P.Batch(node_off, edge_off, src, dst)
        b.plan()
        return {"case": case, "batch": b}
    n = case["n"]
    src, dst = _pairs(case, seed)
    if kind == "count":
        return {"case": case, "src": src, "dst": dst}
    if kind == "csr":
        rowptr, col = _simple_csr(n, src, dst)
        return {"case": case, "rowptr": rowptr, "col": col}
    g = P.Graph(n, src, dst)
    st = {"case": case, "graph": g}
    if kind == "edges":
        # half of the tests are edges of the input, half random pairs
        q, gen = case["queries"], _gen(seed + 1)
        pick = torch.randint(src.numel(), (q,), generator=gen, device=DEV)
        rand = torch.randint(n, (q,), generator=gen, device=DEV, dtype=torch.int32)
        hit = torch.rand(q, generator=gen, device=DEV) < 0.5
        st["u"], st["v"] = src[pick], torch.where(hit, dst[pick], rand)
    elif kind == "serve":
        st["queries"] = _balls(case, seed, src, dst)
        st["server"] = P.Server(g, 6 << 30, slots=2, max_batch_queries=256)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "count":
        o = P.count(case["n"], st["src"], st["dst"])
        return {"T": o["T"], "cc": o["cc"], "total": o["total"], "avg": o["avg"], "m": o["info"]["m"]}
    if kind == "recount":
        return st["graph"].count()
    if kind == "csr":
        g = P.Graph.from_csr(case["n"], st["rowptr"], st["col"], assume_simple_sorted_symmetric=True)
        return g.count()
    if kind == "batch":
        b = P.Batch(*st["args"])
        b.plan()
        return b.run()
    if kind == "batch_run":
        return st["batch"].run()
    if kind == "edges":
        return st["graph"].has_edges(st["u"], st["v"])
    if kind == "core":
        core, top = st["graph"].core(case["k_stop"])
        return {"core": core, "max": top}
    if kind == "cliques":
        return st["graph"].count_k4() if case["k"] == 4 else st["graph"].count_k5()
    srv, done = st["server"], []
    for q, nodes in enumerate(st["queries"]):
        while srv.submit(q, nodes) == P.serve.TRICC_EBUSY:
            done += srv.poll()
    srv.drain()
    done += srv.poll()
    done.sort(key=lambda r: r["qid"])
    return {"triangles": np.array([r["triangles"] for r in done], np.int64),
            "m": np.array([r["m"] for r in done], np.int64),
            "avg": np.array([r["avg_cc"] for r in done], np.float64)}


def work(case):
    """Inputs read once, outputs written once (8 bytes a pair, 12 a node for T
    and cc; 4 bytes a DAG edge or CSR entry plus 8 a node where the graph is
    resident). Set intersections are integer compares: no flops."""
    kind = case["kind"]
    if kind in ("batch", "batch_run"):
        # means of the log-uniform sizes and of the pairs per node (9 in both halves)
        lo, hi = case["nmin"], case["nmax"]
        n = case["graphs"] * (hi - lo) / math.log(hi / lo)
        return {"bytes": n * (12 + 9 * (8 if kind == "batch" else 4)) + 16 * case["graphs"], "flops": 0}
    n, m = case["n"], case["m"]
    if kind == "count":
        b = 8 * m + 12 * n
    elif kind == "recount":
        b = 4 * m + 20 * n
    elif kind == "csr":
        b = 8 * m + 20 * n
    elif kind == "edges":
        b = 9 * case["queries"]
    elif kind == "core":
        b = 8 * m + 12 * n
    elif kind == "cliques":
        b = 4 * m + 8 * n
    else:
        lo, hi = case["kmin"], case["kmax"]
        b = case["queries"] * (4 * (hi - lo) / math.log(hi / lo) + 24)
    return {"bytes": b, "flops": 0}


# ---------------------------------------------------------------------------
# the same results from plain torch, in 64 bits

_MOST_WEDGES = 6_000_000_000


def _count_exact(n, src, dst):
    """Triangles per node and total by enumerating the wedges of the rank
    order and looking their closing edges up; None if there are too many."""
    if not src.numel():
        t = torch.zeros(n, dtype=torch.int64, device=DEV)
        return t, t.clone(), 0
    s, d = src.long(), dst.long()
    key = torch.unique((torch.minimum(s, d) * n + torch.maximum(s, d))[s != d])
    a, b = key // n, key % n
    deg = torch.bincount(a, minlength=n) + torch.bincount(b, minlength=n)
    node = torch.argsort(deg, stable=True)
    rank = torch.empty_like(node)
    rank[node] = torch.arange(n, device=DEV)
    ra, rb = rank[a], rank[b]
    key = torch.sort(torch.minimum(ra, rb) * n + torch.maximum(ra, rb))[0]
    lo, hi = key // n, key % n
    end = torch.cumsum(torch.bincount(lo, minlength=n), 0)
    later = end[lo] - 1 - torch.arange(lo.numel(), device=DEV)  # wedges that begin with each edge
    cum = torch.cumsum(later, 0)
    wedges = int(cum[-1]) if cum.numel() else 0
    if wedges > _MOST_WEDGES:
        return None
    T = torch.zeros(n, dtype=torch.int64, device=DEV)
    e0, done = 0, 0
    while e0 < lo.numel():
        e1 = max(e0 + 1, int(torch.searchsorted(cum, done + (1 << 26), right=True)))
        w = later[e0:e1]
        base = cum[e0:e1] - w - done
        i = torch.repeat_interleave(torch.arange(e0, e1, device=DEV), w)
        j = i + 1 + torch.arange(i.numel(), device=DEV) - base[i - e0]
        want = hi[i] * n + hi[j]
        at = torch.searchsorted(key, want)
        hit = key[torch.clamp(at, max=key.numel() - 1)] == want
        i, j = i[hit], j[hit]
        for x in (lo[i], hi[i], hi[j]):
            T += torch.bincount(x, minlength=n)
        done, e0 = int(cum[e1 - 1]), e1
    out = torch.empty_like(T)
    out[node] = T
    return deg, out, int(T.sum()) // 3


def _cc(deg, T):
    d = deg.double()
    return torch.where(deg >= 2, 2.0 * T.double() / torch.clamp(d * (d - 1.0), min=1.0), torch.zeros_like(d))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("edges", "core", "cliques"):
        return None  # whole numbers only
    if kind in ("batch", "batch_run"):
        node_off, edge_off, src, dst = _batch_pairs(case, seed)
        n_of, m_of = np.diff(node_off), np.diff(edge_off)
        shift = torch.repeat_interleave(torch.from_numpy(node_off[:-1]).to(DEV), torch.from_numpy(m_of).to(DEV))
        if shift.numel() > 100_000_000:
            return None
        got = _count_exact(int(node_off[-1]), src.long() + shift, dst.long() + shift)
        if got is None:
            return None
        deg, T, total = got
        of = torch.repeat_interleave(torch.arange(case["graphs"], device=DEV), torch.from_numpy(n_of).to(DEV))
        cc = _cc(deg, T)
        tri = torch.zeros(case["graphs"], dtype=torch.int64, device=DEV).index_add_(0, of, T) // 3
        avg = torch.zeros(case["graphs"], dtype=torch.float64, device=DEV).index_add_(0, of, cc)
        return {"T": T, "cc": cc, "graph_tri": tri, "graph_avg": avg / torch.from_numpy(n_of).to(DEV),
                "batch_tri": torch.tensor([total])}
    n = case["n"]
    if case["m"] > 20_000_000:
        return None
    src, dst = _pairs(case, seed)
    if kind == "serve":
        tri, ms, avg = [], [], []
        s, d = src.long(), dst.long()
        key = torch.unique((torch.minimum(s, d) * n + torch.maximum(s, d))[s != d])
        a, b = key // n, key % n
        local = torch.full((n,), -1, dtype=torch.int64, device=DEV)
        wedges_left = True
        for nodes in _balls(case, seed, src, dst):
            v = torch.from_numpy(nodes).to(DEV).long()
            local[v] = torch.arange(v.numel(), device=DEV)
            x, y = local[a], local[b]
            inside = (x >= 0) & (y >= 0)
            got = _count_exact(v.numel(), x[inside], y[inside])
            local[v] = -1
            if got is None:
                wedges_left = False
                break
            tri.append(got[2])
            ms.append(int(inside.sum()))
            avg.append(float(_cc(got[0], got[1]).mean()))
        if not wedges_left:
            return None
        return {"triangles": np.array(tri, np.int64), "m": np.array(ms, np.int64), "avg": np.array(avg)}
    got = _count_exact(n, src, dst)
    if got is None:
        return None
    deg, T, total = got
    cc = _cc(deg, T)
    out = {"T": T, "cc": cc, "total": torch.tensor([total]), "avg": cc.mean().reshape(1)}
    if kind == "count":
        out["m"] = int(deg.sum()) // 2
    return out
