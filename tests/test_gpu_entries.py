"""GPU parity of the traversals over the entry views (matrices whose entries
sit in short COO blocks) against the oracle.

Pull streams the row-entry view in chunks of 256 entries, 64 per wave step,
64 queued hits at a time, with an LDS bitmap of x that folds 2^f columns into
a bit above 2^20 columns; push walks the listed columns.  The sizes are the
edges of those units; the tolerance is the suite's 1e-5 * sum |a_ij x_j|
(the sums are fp64, so only the products' and the result's rounding remain).
"""
import numpy as np
import pytest

import oracle
import paper_2608_16308_amd as dbs
import workloads as wl
from gpu_helpers import REL_TOL, check_spmspv, gpu_matrix, log, mask_words, oracle_matrix, to_dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def list_matrix(m, n, nnz, key, dtype=np.float32, long_row=0):
    """nnz entries in random rows (many rows empty), `long_row` of them in one
    row; columns at least 16 apart where the row allows it, so that the blocks
    are COO blocks of one or two entries."""
    rng = wl.rng_for(wl.W_RAND, 91, key, nnz)
    rows = rng.integers(0, m, nnz)
    if long_row:
        rows[:long_row] = m // 2
    ent = np.unique(rows.astype(np.int64) * n + rng.integers(0, n, nnz))
    while ent.size < nnz:
        ent = np.unique(np.concatenate([ent, rng.integers(0, m, nnz).astype(np.int64) * n + rng.integers(0, n, nnz)]))
    ent = np.sort(rng.permutation(ent)[:nnz])
    vals = None if dtype is None else wl._nonzero_uniform(wl.rng_for(wl.W_RAND, 92, key), -1.0, 1.0, nnz, dtype=dtype)
    return wl.csr_from_coo(m, n, ent // n, ent % n, vals)


def x_of(n, k, key, dtype=np.float32):
    idx = np.sort(wl.rng_for(wl.W_RAND, 93, key, k).choice(n, min(k, n), replace=False)).astype(np.int32)
    return idx, wl._nonzero_uniform(wl.rng_for(wl.W_RAND, 94, key), -1.0, 1.0, idx.size, dtype=dtype)


@pytest.mark.parametrize("nnz,long_row", [(1, 0), (63, 0), (64, 60), (65, 0), (255, 200), (256, 0), (257, 257),
                                          (4096, 3000), (16385, 0), (70000, 9000)])
def test_chunk_edges(torch, nnz, long_row):
    for dt in (np.float32, np.float16, None):
        a = list_matrix(3000, 20000, nnz, 1, dt, long_row)
        A, om = gpu_matrix(a), oracle_matrix(a)
        assert A.info()["blocks_by_type"]["coo"] == A.info()["nblk"]
        ctx = dbs.Context(A)
        mw = mask_words(wl.rng_for(wl.W_RAND, 95, nnz).random(a.m) < 0.5)
        sr = "or_and" if dt is None else "plus_times"
        # one index, few, many (more than a vector block holds one of), all
        for k in (1, 40, 1500, 3000, 20000):
            xi, xv = x_of(a.n, k, 2, dt or np.float32)
            for p in ("push", "pull", "auto"):
                label = f"entries nnz={nnz} {dt} k={k} path={p}"
                log(label)
                check_spmspv(ctx, A, om, a, xi, xv.astype(np.float64), path=p, semiring=sr, label=label)
            check_spmspv(ctx, A, om, a, xi, xv.astype(np.float64), path="pull", semiring=sr, mask=mw, complement=True,
                         label=f"entries nnz={nnz} {dt} k={k} masked pull")
            check_spmspv(ctx, A, om, a, xi, xv.astype(np.float64), path="push", semiring=sr, mask=mw,
                         label=f"entries nnz={nnz} {dt} k={k} masked push")


@pytest.mark.parametrize("n", [(1 << 20) - 3, (1 << 20) + 1, 2_000_003, 3_000_001, 9_000_017])
def test_folded_bitmap(torch, n):
    """Columns that share a bitmap bit with a listed one are not listed: rows
    that only they reach stay out of y."""
    a = list_matrix(700, n, 30000, 3)
    x_all = np.unique(a.col_idx)
    near = np.unique(np.concatenate([np.clip(x_all[::3] + d, 0, n - 1) for d in (-3, -1, 1, 2)]))
    near = np.setdiff1d(near, x_all).astype(np.int32)          # neighbours of stored columns only
    real = x_all[1::7].astype(np.int32)
    A, om = gpu_matrix(a), oracle_matrix(a)
    ctx = dbs.Context(A)
    for name, xi in (("near only", near), ("near and real", np.sort(np.concatenate([near, real])))):
        xv = wl._nonzero_uniform(wl.rng_for(wl.W_RAND, 96, xi.size), -1.0, 1.0, xi.size)
        for sr in ("plus_times", "or_and"):
            for p in ("pull", "auto"):
                label = f"folded n={n} {name} {sr} path={p}"
                log(label)
                st = check_spmspv(ctx, A, om, a, xi, xv, path=p, semiring=sr, label=label)
                assert name != "near only" or st["y_nnz"] == 0


def test_unsorted_rows(torch):
    """Columns in any order within a row of the input."""
    a = list_matrix(500, 9000, 20000, 4, long_row=3000)
    rng = wl.rng_for(wl.W_RAND, 97, 0)
    col, val = a.col_idx.copy(), a.vals.copy()
    for i in range(a.m):
        s = slice(a.row_ptr[i], a.row_ptr[i + 1])
        o = rng.permutation(a.row_ptr[i + 1] - a.row_ptr[i])
        col[s], val[s] = col[s][o], val[s][o]
    b = wl.CSR(a.m, a.n, a.row_ptr, col, val)
    A, om = gpu_matrix(b), oracle_matrix(a)
    ctx = dbs.Context(A)
    xi, xv = x_of(a.n, 900, 5)
    for p in ("push", "pull", "auto"):
        check_spmspv(ctx, A, om, a, xi, xv, path=p, label=f"unsorted rows path={p}")


@pytest.mark.parametrize("k", [60, 2500])
def test_repeated_indices_count_once(torch, k):
    """Repeats anywhere in the list (next to each other, within a wave, across
    waves; runs of one 32-column word interrupted by another) add nothing."""
    a = list_matrix(2000, 50000, 60000, 6)
    A, om = gpu_matrix(a), oracle_matrix(a)
    ctx = dbs.Context(A)
    xi, xv = x_of(a.n, k, 7)
    xi[:4] = [64, 65, 7000, 66] if not np.isin([64, 65, 7000, 66], xi[4:]).any() else xi[:4]
    rng = wl.rng_for(wl.W_RAND, 98, k)
    rep = rng.integers(0, k, k // 3)
    order = rng.permutation(k + rep.size)
    yi = np.concatenate([xi, xi[rep]])[order]
    yv = np.concatenate([xv, xv[rep]])[order]
    yi, yv = np.concatenate([yi[:1], yi]), np.concatenate([yv[:1], yv])
    ri, rv, rs = om.spmspv(xi, xv.astype(np.float64))
    for p in ("push", "pull", "auto"):
        log(f"repeated indices k={k} path={p}")
        y_idx, y_val, st = ctx.spmspv(A, to_dev(yi.astype(np.int32)), to_dev(yv), path=p, stats=True)
        torch.cuda.synchronize()
        assert st["error_flags"] == 2
        assert st["n_nzblk"] == np.unique(xi >> 4).size
        assert np.array_equal(y_idx.cpu().numpy(), ri)
        assert oracle.within_tol(y_val.cpu().numpy(), rv, rs, REL_TOL).all()


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("m,n,keep", [(16, 16, 0.004), (37, 1500, 0.02), (1000, 129, 0.03), (513, 4099, 0.02),
                                      (40, 16400, 0.05)])
def test_views_of_a_device_built_matrix(torch, dtype, m, n, keep):
    """The device construction counts and fills the same views: sparse and
    dense x on both paths, with empty rows, against the oracle."""
    rng = wl.rng_for(wl.W_RAND, 99, m, n)
    w = np.where(rng.random((m, n)) < keep, rng.uniform(0.1, 1.0, (m, n)), 0.0).astype(dtype)
    w[m // 3:m // 2] = 0
    w[m - 1, n - 1] = 0.5
    r, c = np.nonzero(w)
    a = wl.csr_from_coo(m, n, r, c, w[r, c])
    A, om = dbs.Matrix.from_dense(to_dev(w)), oracle_matrix(a)
    ctx = dbs.Context(A)
    for k in (1, 7, n // 8 + 1, n):
        xi, xv = x_of(n, k, 7, dtype)
        for p in ("push", "pull", "auto"):
            log(f"device-built {dtype.__name__} {m}x{n} k={k} path={p}")
            check_spmspv(ctx, A, om, a, xi, xv.astype(np.float64), path=p, label=f"device-built {m}x{n} k={k} {p}")
        x = np.zeros(n, dtype)
        x[xi] = xv
        y32 = torch.empty(m, dtype=torch.float32, device="cuda:0")
        ctx.spmspv_dense(A, to_dev(x), y32=y32)
        torch.cuda.synchronize()
        ri, rv, rs = om.spmspv(xi, xv.astype(np.float64))
        y64, S = np.zeros(m), np.zeros(m)
        y64[ri], S[ri] = rv, rs
        assert oracle.within_tol(y32.cpu().numpy(), y64, S, REL_TOL).all()


def test_large_matrix_of_many_entry_blocks(torch):
    """16M entries in COO blocks of 24: pull goes over the blocks, push over
    the listed columns, in turn on one context."""
    rng = wl.rng_for(wl.W_RAND, 97, 0)
    nbr, nbc, per, fill = 1024, 4099, 680, 24
    J = np.argsort(rng.random((nbr, nbc)), axis=1)[:, :per]
    cell = (rng.integers(0, 256, (nbr, per, 1)) + (2 * rng.integers(0, 128, (nbr, per, 1)) + 1) * np.arange(fill)) & 255
    n = nbc * 16
    key = np.sort((((np.arange(nbr)[:, None, None] * 16 + cell // 16) * n) + J[:, :, None] * 16 + cell % 16).reshape(-1))
    a = wl.csr_from_coo(nbr * 16, n, key // n, key % n, wl._nonzero_uniform(rng, -1.0, 1.0, key.size, dtype=np.float32))
    A, om = gpu_matrix(a), oracle_matrix(a)
    i = A.info()
    assert i["blocks_by_type"]["coo"] == i["nblk"] and i["nnz"] > max(15 << 20, 2 * i["nblk"])
    ctx = dbs.Context(A)
    mw = mask_words(rng.random(a.m) < 0.5)
    for k in (1, 30, 300, 5000, 60000):
        xi, xv = x_of(n, k, 3)
        for sr in ("plus_times", "or_and"):
            for p in ("pull", "push", "auto"):
                label = f"many-entry blocks k={k} {sr} {p}"
                log(label)
                check_spmspv(ctx, A, om, a, xi, xv.astype(np.float64), path=p, semiring=sr, mask=mw, complement=True, label=label)


@pytest.mark.parametrize("dtype,m,n", [(np.float32, 12003, 30017), (np.float16, 12000, 30016)])
def test_dense_activation_on_many_entries(torch, dtype, m, n):
    """More than 20M entries in short COO blocks: the scan chooses between the
    stream and push; nearly empty activations (push) and others in turn."""
    g = torch.Generator(device="cuda").manual_seed(5)
    dt = torch.float32 if dtype == np.float32 else torch.float16
    w = torch.where(torch.rand((m, n), device="cuda", generator=g) < 0.065,
                    torch.rand((m, n), device="cuda", generator=g) - 0.5, torch.zeros((), device="cuda")).to(dt)
    A = dbs.Matrix.from_dense(w)
    i = A.info()
    assert i["nnz"] > 20 << 20 and i["nnz"] < 32 * i["nblk"]
    ctx = dbs.Context(A)
    w64 = w.double()
    taken = set()
    for active in (0.0003, 0.2, 0.02, 0.0003, 0.0, 1.0):
        x = (torch.randn(n, device="cuda", generator=g) * (torch.rand(n, device="cuda", generator=g) < active)).to(dt)
        ref, S = w64 @ x.double(), w64.abs() @ x.double().abs()
        for path in ("auto", "pull"):
            log(f"dense on many entries {dtype.__name__} {m}x{n} active={active} {path}")
            for stats in (False, True):
                y32 = torch.full((m,), -7.0, device="cuda")
                out = ctx.spmspv_dense(A, x, y32=y32, path=path, stats=stats)
                torch.cuda.synchronize()
                y = out[0] if stats else out
                if stats and path == "auto":
                    taken.add(out[1]["path"])
                assert bool(((y32.double() - ref).abs() <= REL_TOL * S).all())
                assert torch.equal(y, y32) if dtype == np.float32 else bool(((y.double() - ref).abs() <= 2.0 ** -10 * ref.abs() + 2.0 ** -24).all())
    assert taken == {"push", "pull"}
