"""The bytes model of calls over the entry views, against counts taken entry
by entry."""
import numpy as np
import pytest

import paper_2608_16308_amd as dbs
import workloads as wl
from paper_2608_16308_amd.bytes_model import BytesModel


@pytest.mark.parametrize("k", [1, 40, 300, 1500])
@pytest.mark.parametrize("path", ["push", "pull"])
def test_entry_view_bytes(path, k):
    n = 5000
    rng = wl.rng_for(wl.W_RAND, 140, k)
    key = np.unique(rng.integers(0, n, 20000) * n + rng.integers(0, n, 20000))
    a = wl.csr_from_coo(n, n, key // n, key % n, np.ones(key.size, np.float32))
    hm = dbs.HostMatrix.from_csr(a.m, a.n, a.row_ptr, a.col_idx, a.vals)
    model = BytesModel(a.m, a.n, a.row_ptr, a.col_idx, hm.arrays(), hm.info(), 4)
    x = np.sort(rng.choice(n, k, replace=False))
    r = model.call(x, path)
    nbc = (n + 15) // 16
    if path == "push" and k > nbc:  # (no item list that long: over the blocks)
        assert not r["views"] and r["bytes_main"] == model.call(x, path, blocks=True)["bytes_main"]
        return
    assert r["views"]
    hit = np.isin(key % n, x)
    rows = np.unique(key[hit] // n)
    entries, words = int(hit.sum()), np.unique(rows // 32).size
    assert r["useful_nnz"] == entries and r["y_nnz"] == rows.size
    common = 8 * rows.size + 4 * words
    if path == "push":
        listed = np.unique(key[hit] % n).size
        assert r["bytes_main"] == common + 16 * listed + entries * 8
        assert r["bytes_blocker"] == k * 16 + 8 * k + 16 * listed
    else:
        assert r["bytes_main"] == common + 4 * key.size + 4 * -(-key.size // 256) + 2 * nbc + entries * 4 + 4 * k + 4 * rows.size
        assert r["bytes_blocker"] == k * 16
    assert r["bytes_scan"] == 0
    assert r["bytes_total"] == r["bytes_blocker"] + r["bytes_main"] + r["bytes_finalize"]
