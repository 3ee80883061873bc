"""GPU: offsets, bins and in-list items of the built DAG at the edges of the
layout passes' tiles (1,024 nodes; more per tile above 2^20 nodes), against the
same quantities formed with numpy from the DAG's own arrays."""
import numpy as np
import pytest
import torch

import oracle
import paper_1606_07550_amd as P
from paper_1606_07550_amd import inputs as I

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
