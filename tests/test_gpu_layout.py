"""GPU: offsets, bins and in-list items of the built DAG at the edges of the
layout passes' tiles (1,024 nodes; more per tile above 2^20 nodes), against the
same quantities formed with numpy from the DAG's own arrays."""
import numpy as np
import pytest
import torch

import oracle
import paper_1606_07550_amd as P
from paper_1606_07550_amd import _native

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [1, 63, 1023, 1024, 1025, 2049, 70_001, (1 << 20) - 1, (1 << 20) + 1])
def test_layout_tiles(n):
    rng = np.random.default_rng(n)
    m = min(20 * n, 400_000)
    s = rng.integers(0, n, m, dtype=np.int32)
    d = (rng.random(m) ** 3 * n).astype(np.int32)  # a few heavy nodes: every bin but the hubs'
    tuning = {"bin_limit": [4, 8, 16, 64, 4096], "bin_variant": [21, 22, 23, 24, 14, 9], "min_side": 1}
    g = P.Graph(n, torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV), tuning=tuning)
    out = g.count()
    torch.cuda.synchronize()
    a, info = g.arrays(), g.info
    doff, deg = a["doff"].cpu().numpy(), a["deg"].cpu().numpy()
    p = np.diff(doff)
    assert doff[0] == 0 and doff[-1] == info["m"]
    assert info["max_deg"] == deg.max(initial=0) and info["max_outdeg"] == p.max(initial=0)
    assert info["n_deg2"] == int((deg >= 2).sum())
    lim = np.array(tuning["bin_limit"])
    b = np.searchsorted(lim, p)
    assert list(info["bin_count"]) == [int(((b == q) & (p >= 2)).sum()) for q in range(6)]
    cap = np.array([P.variant_capacity(v) for v in tuning["bin_variant"]])
    din = deg - p
    own = (p >= 3) & (din >= 1) & (p <= 4096)
    items = -(-din // cap[b])
    assert list(info["bin_in_items"]) == [int(items[own & (b == q)].sum()) for q in range(6)]
    ref = oracle.count(n, s, d)
    np.testing.assert_array_equal(out["T"].cpu().numpy().view(np.uint64), ref["T"])
    assert g.count_check() == (ref["total"], 3 * ref["total"])


def _parity(n, s, d):
    g = P.Graph(n, torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV))
    out = g.count()
    torch.cuda.synchronize()
    ref = oracle.count(n, s, d)
    np.testing.assert_array_equal(out["T"].cpu().numpy().view(np.uint64), ref["T"])
    assert g.info["m"] == ref["m"]
    a = g.arrays()
    off, deg = a["off"].cpu().numpy(), a["deg"].cpu().numpy()
    loops = s == d
    raw = np.bincount(s[~loops], minlength=n) + np.bincount(d[~loops], minlength=n)
    np.testing.assert_array_equal(np.diff(off), raw)
    assert off[0] == 0 and int(deg.sum()) == 2 * ref["m"]


# a chunk of the row passes holds 2**18 entries (two per pair): one chunk per
# partition, the last size with one, the first with two, several, and
# partitions without an entry before, between and after the others
@pytest.mark.parametrize("n,lo,hi,m", [(5000, 0, 5000, 1000), (5000, 3000, 3100, 5000), (9000, 0, 900, 1 << 17),
                                       (9000, 0, 900, (1 << 17) + 1), (70_000, 40_000, 40_900, 500_000),
                                       (1024, 0, 1024, 1 << 17), (1025, 0, 1025, 300_000)])
def test_partition_chunks(n, lo, hi, m):
    rng = np.random.default_rng(m + n)
    s, d = (rng.integers(lo, hi, m, dtype=np.int32) for _ in range(2))
    _parity(n, s, d)


@pytest.mark.parametrize("n,deg", [(1, 0), (64, 0), (300, 5), (1000, 255), (1000, 64)])
def test_csr_rows_checked_everywhere(n, deg):
    """Trusted rows: accepted as they are; one wrong entry anywhere, or wrong
    bounds, is refused with the status of its kind."""
    rng = np.random.default_rng(deg)
    m = n * deg // 2
    s, d = (rng.integers(0, n, m, dtype=np.int32) for _ in range(2))
    rowptr, col = oracle_csr(n, s, d)
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    g = P.Graph.from_csr(n, dev(rowptr), dev(col), assume_simple_sorted_symmetric=True)
    assert g.info["m"] == col.size // 2

    def refused(rp, cl, status):
        with pytest.raises(P.TriccError) as e:
            P.Graph.from_csr(n, dev(rp), dev(cl), assume_simple_sorted_symmetric=True)
        assert e.value.status == status

    EINVAL, ERANGE = 1, 2
    bad = rowptr.copy()
    bad[-1] += 1
    refused(bad, col, EINVAL)
    if not col.size:
        return
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    inner = np.flatnonzero(np.diff(rows) == 0) + 1  # entries with a predecessor in their row
    for i in inner[[0, inner.size // 2, -1]]:
        c = col.copy()
        c[i] = c[i - 1]
        refused(rowptr, c, EINVAL)
    for i in (0, col.size // 2, col.size - 1):
        c = col.copy()
        c[i] = n
        refused(rowptr, c, ERANGE)
        c[i] = -1
        refused(rowptr, c, ERANGE)
    v = int(np.flatnonzero(np.diff(rowptr))[-1])  # the last row's own id in its place
    r = np.unique(np.concatenate([col[rowptr[v]:rowptr[v + 1]][1:], [v]])).astype(np.int32)
    c = col.copy()
    c[rowptr[v]:rowptr[v] + r.size] = r
    refused(rowptr, c, EINVAL)
    bad = rowptr.copy()
    bad[n // 2] = col.size + 5
    refused(bad, col, EINVAL)


@pytest.mark.parametrize("n", [3, 700, 600_000])
def test_csr_steps_down_inside_rows(n):
    """Trusted rows whose starts all fall (every row ends above the next row's
    first id), rise, or both: one fall inside a row is found, wherever it is."""
    r = np.random.default_rng(n)
    ring = np.arange(n)
    far = r.permutation(n)
    s, d = np.concatenate([ring, far[:n // 2]]), np.concatenate([(ring + 1) % n, far[n - n // 2:]])
    rowptr, col = oracle_csr(n, s, d)
    dev = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    P.Graph.from_csr(n, dev(rowptr), dev(col), assume_simple_sorted_symmetric=True)
    path = np.stack([ring[:-1], ring[1:]])  # rows {v - 1, v + 1}: every start from row 2 on falls
    rp, cl = oracle_csr(n, *path)
    P.Graph.from_csr(n, dev(rp), dev(cl), assume_simple_sorted_symmetric=True)
    for rowptr, col in ((rowptr, col), (rp, cl)):
        for v in (np.flatnonzero(np.diff(rowptr) > 1)[k] for k in (0, -1)):
            c = col.copy()
            c[rowptr[v]:rowptr[v] + 2] = c[rowptr[v]:rowptr[v] + 2][::-1]
            with pytest.raises(P.TriccError) as e:
                P.Graph.from_csr(n, dev(rowptr), dev(c), assume_simple_sorted_symmetric=True)
            assert e.value.status == 1


def oracle_csr(n, s, d):
    keep = s != d
    a = np.concatenate([s[keep], d[keep]]).astype(np.int64)
    b = np.concatenate([d[keep], s[keep]]).astype(np.int64)
    key = np.unique(a * n + b)
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=rowptr[1:])
    return rowptr, (key % n).astype(np.int32)


@pytest.mark.parametrize("n", [40_000, 1 << 18, (1 << 18) + 1, 1 << 20, (1 << 20) + 1, 3 * (1 << 20) + 5])
def test_long_rows(n):
    """Rows at the edges of the sort classes, with repeats, below and above
    the widths of the bitmaps: sorted and unique in the built graph."""
    rng = np.random.default_rng(n)
    lens = [2, 8, 9, 64, 65, 1024, 1025, 4096, 4097, 8192, 8193, 16_384, 16_385, 32_768, 32_769, 70_001]
    hubs = np.concatenate([[0, n - 1], rng.choice(np.arange(1, n - 1), len(lens) - 2, replace=False)])
    want, s, d = {}, [], []
    for h, k in zip(hubs, lens):
        others = np.setdiff1d(np.arange(n, dtype=np.int32), hubs.astype(np.int32))
        lo, hi = (0, others.size) if k % 2 else (others.size // 3, others.size // 3 + 3 * k)  # spread or dense
        w = others[rng.integers(lo, min(hi, others.size), k)]
        w[:2] = others[[0, -1]][:k]
        flip = rng.random(k) < 0.5
        s.append(np.where(flip, h, w))
        d.append(np.where(flip, w, h))
        want[int(h)] = np.unique(w)
    s, d = np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32)
    mix = rng.permutation(s.size)
    s, d = s[mix], d[mix]
    g = P.Graph(n, torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV))
    a = g.arrays()
    off, deg, adj = (a[k].cpu().numpy() for k in ("off", "deg", "adj"))
    for h, w in want.items():
        assert deg[h] == w.size
        np.testing.assert_array_equal(adj[off[h]:off[h] + deg[h]], w)
    assert g.info["large_rows"] == 2
    out = g.count()
    ref = oracle.count(n, s, d)
    np.testing.assert_array_equal(out["T"].cpu().numpy().view(np.uint64), ref["T"])
    assert int(deg.sum()) == 2 * ref["m"]


@pytest.mark.parametrize("outer", [1500, 2725, 2735, 5460, 5475, 9000])
def test_in_list_parts(outer):
    """Owners with more in-neighbours than a table kernel takes lists at a
    time: chunks of 4,096 in-neighbours in parts of 2,048 (the large-table
    variant on a graph whose out-degrees fit the smaller table)."""
    rng = np.random.default_rng(outer)
    core = 48
    i, j = np.triu_indices(core, 1)
    s, d = [i], [j]
    for v in range(core, core + outer):  # each outer node meets 36 of the 48 core nodes, and two outer ones
        s.append(np.full(38, v))
        d.append(np.concatenate([rng.choice(core, 36, replace=False), rng.integers(core, core + outer, 2)]))
    s, d = np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32)
    n = core + outer
    perm = rng.permutation(n).astype(np.int32)
    s, d = perm[s], perm[d]
    tuning = {"bin_limit": [2, 3, 4, 5, 4096], "bin_variant": [21, 23, 24, 20, 14, 9], "min_side": 1}
    g = P.Graph(n, torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV), tuning=tuning)
    out = g.count()
    ref = oracle.count(n, s, d)
    np.testing.assert_array_equal(out["T"].cpu().numpy().view(np.uint64), ref["T"])
    assert g.count_check() == (ref["total"], 3 * ref["total"])


@pytest.mark.parametrize("n", [1000, 1024, 1025, 3000])
@pytest.mark.parametrize("m", [1, 8191, 8192, 8193])
def test_pairs_of_one_tile_and_of_two(n, m):
    """One partition and several; pairs in one tile, where the sizes come from
    the placing itself, and in two; ids that share a partition along a wavefront
    and ids that do not; an id out of range is refused in every case."""
    rng = np.random.default_rng(n + m)
    for ordered in (False, True):
        s = rng.integers(0, n, m).astype(np.int32)
        d = rng.integers(0, n, m).astype(np.int32)
        if ordered:
            s = np.sort(s)
        g = P.Graph(n, torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV))
        out = g.count()
        torch.cuda.synchronize()
        ref = oracle.count(n, s, d, order=1)
        np.testing.assert_array_equal(out["T"].cpu().numpy().view(np.uint64), ref["T"])
        assert g.info["m"] == ref["m"]
    for bad in (-1, n):
        e = d.copy()
        e[m // 2] = bad
        for a, b in ((s, e), (e, s)):
            with pytest.raises(_native.TriccError) as ei:
                P.Graph(n, torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV))
            assert ei.value.status == _native.TRICC_ERANGE


@pytest.mark.parametrize("ranges", [16, 17, 32, 33, 96])
def test_long_rows_of_many_ids(ranges):
    """Rows on both sides of the bound between bitmaps and networks or merges
    (1,024 entries per 2^20 ids above 16 such ranges), with repeats, of graphs
    of up to 10^8 ids: sorted and unique in the built graph."""
    n = (ranges << 20) - 3
    bound = 1024 * ranges
    lens = sorted({16_384, 16_385, 32_767, 32_768, 32_769, 65_536, 65_537, bound - 1, bound, bound + 1, 100_001})
    rng = np.random.default_rng(ranges)
    hubs = np.sort(rng.choice(n, len(lens), replace=False)).astype(np.int64)
    hubs[0], hubs[-1] = 0, n - 1
    s, d, want = [], [], []
    for i, (h, k) in enumerate(zip(hubs, lens)):
        w = rng.integers(0, n, k) if i % 2 else n // 3 + rng.integers(0, 2 * k, k)  # spread or in one range
        w = np.where(np.isin(w, hubs), 5, w)
        flip = rng.random(k) < 0.5
        s.append(np.where(flip, h, w))
        d.append(np.where(flip, w, h))
        want.append(np.unique(w))
    s, d = np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32)
    mix = rng.permutation(s.size)
    g = P.Graph(n, torch.from_numpy(s[mix]).to(DEV), torch.from_numpy(d[mix]).to(DEV))
    a = g.arrays()
    at = torch.from_numpy(hubs).to(DEV)
    off, deg = a["off"][at].cpu().numpy(), a["deg"][at].cpu().numpy()
    for o, k, w in zip(off, deg, want):
        assert k == w.size
        np.testing.assert_array_equal(a["adj"][int(o):int(o) + int(k)].cpu().numpy(), w)
    assert g.info["large_rows"] == sum(k > 32_768 for k in lens)
    assert int(a["deg"].sum()) == 2 * g.info["m"] == 2 * sum(w.size for w in want)


def test_more_short_rows_than_a_launch_has_blocks():
    """A ring of 40 million nodes, each joined to the two after it: rows of 4
    entries in 1.25 million blocks, more than the row sort launches at once."""
    n = 40_000_000
    i = torch.arange(n, device=DEV, dtype=torch.int32)
    d = torch.cat([(i + 1) % n, (i + 2) % n])
    mix = torch.randperm(2 * n, device=DEV)
    g = P.Graph(n, i.repeat(2)[mix].contiguous(), d[mix].contiguous())
    a = g.arrays()
    assert bool((a["deg"] == 4).all()) and bool((a["off"] == 4 * torch.arange(n + 1, device=DEV)).all())
    rows = a["adj"].view(n, 4)
    want = torch.sort(torch.stack([(i + k) % n for k in (-2, -1, 1, 2)], 1), 1)[0]
    assert bool((rows == want).all())
    out = g.count()
    assert bool((out["T"] == 3).all()) and int(out["total"]) == n


@pytest.mark.parametrize("n", [1, 1024, 1025, 70_001, (1 << 20) + 1])
def test_new_bins_of_the_same_dag(n):
    """Retuning forms the node bins and in-list items anew and nothing else: the
    offsets, which a count or query on another stream may be reading, are not
    written (marked here, and put back before the count)."""
    rng = np.random.default_rng(n)
    m = min(20 * n, 400_000)
    s = rng.integers(0, n, m, dtype=np.int32)
    d = (rng.random(m) ** 3 * n).astype(np.int32)
    g = P.Graph(n, torch.from_numpy(s).to(DEV), torch.from_numpy(d).to(DEV))
    a, info = g.arrays(), g.info
    doff = a["doff"].clone()
    a["doff"].fill_(-5)
    lim, var = [4, 8, 16, 64, 4096], [21, 22, 23, 24, 14, 9]
    g.retune({"bin_limit": lim, "bin_variant": var, "min_side": 1})
    assert bool((a["doff"] == -5).all())
    a["doff"].copy_(doff)
    now = g.info
    assert all(now[k] == info[k] for k in ("m", "max_deg", "max_outdeg", "n_deg2"))
    p, deg = np.diff(doff.cpu().numpy()), a["deg"].cpu().numpy()
    b = np.searchsorted(np.array(lim), p)
    assert list(now["bin_count"]) == [int(((b == q) & (p >= 2)).sum()) for q in range(6)]
    items = -(-(deg - p) // np.array([P.variant_capacity(v) for v in var])[b])
    own = (p >= 3) & (deg - p >= 1) & (p <= 4096)
    assert list(now["bin_in_items"]) == [int(items[own & (b == q)].sum()) for q in range(6)]
    ref = oracle.count(n, s, d)
    np.testing.assert_array_equal(g.count()["T"].cpu().numpy().view(np.uint64), ref["T"])


@pytest.mark.parametrize("run", [1, 3, 15, 16, 17, 64, 5000])
@pytest.mark.parametrize("n", [2000, 300_000])
def test_runs_of_equal_pairs(n, run):
    """Rows sorted by bitmap whose entries come in runs of one id, id 0 and the
    highest among them."""
    rng = np.random.default_rng(run)
    ids = np.concatenate([[0, n - 1, 0, 1, 2], rng.integers(0, n, 6000 // run), [0, n - 1]])
    ids = ids[ids != 7]
    w = np.repeat(ids, run)
    w = np.concatenate([w, np.full(max(0, 5000 - w.size), 0)]).astype(np.int32)
    g = P.Graph(n, torch.full((w.size,), 7, dtype=torch.int32, device=DEV), torch.from_numpy(w).to(DEV))
    a = g.arrays()
    want = np.unique(w)
    off, deg = int(a["off"][7]), int(a["deg"][7])
    np.testing.assert_array_equal(a["adj"][off:off + deg].cpu().numpy(), want)
    assert g.info["m"] == want.size
    np.testing.assert_array_equal(torch.nonzero(a["deg"] == 1).flatten().cpu().numpy(), want)
