"""GPU parity of the matrix-core pass for dense activations (one to eight)
against the oracle: every block class (Dense, row formats, COO in the
descriptor and in a record, ForceCSC, row formats of more than 128 entries),
ragged shapes, one workgroup and several per block row (block rows of more
than 128 blocks), infinities and NaN in A and x, fp16 subnormals.

fp16 outputs within one ulp of the fp64 sum's rounding; fp32 within the
suite's 1e-5 * sum |a_ij x_j| (a block's 16 products are summed in fp32, the
blocks in fp64)."""
import numpy as np
import pytest

import oracle
import paper_2608_16308_amd as dbs
import workloads as wl
from gpu_helpers import REL_TOL, check_f16, gpu_matrix, log, oracle_matrix, to_dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def check(ctx, A, om, X, label):
    """Y = A X for the rows of X, through the batched and the one-vector call."""
    torch = torch_mod()
    log(label)
    nb = X.shape[0]
    refs = [oracle_sums(om, X[b]) for b in range(nb)]
    # every call finds what the ones before left in the scratch; without
    # statistics nothing but the pass itself restores it
    for stats in (False, False, True, False):
        Y32 = torch.full((nb, om.m), -7.0, dtype=torch.float32, device="cuda:0")
        if nb == 1:
            out = ctx.spmspv_dense(A, to_dev(X[0]), y32=Y32[0], stats=stats)
        else:
            out = ctx.spmm_dense(A, to_dev(X), Y32=Y32, stats=stats)
        torch.cuda.synchronize()
        Y, st = out if stats else (out, None)
        Y = Y[None] if nb == 1 else Y
        blocks = np.unique(np.nonzero((X != 0).any(0))[0] >> 4)
        assert st is None or st["n_nzblk"] == blocks.size, (label, st)
        for b in range(nb):
            y64, S = refs[b]
            g, g32 = Y[b].cpu().numpy(), Y32[b].cpu().numpy()
            if X.dtype == np.float16:
                check_f16(g, y64, f"{label} vector {b}")
            else:
                assert oracle.within_tol(g, y64, S, REL_TOL).all(), f"{label} vector {b}"
            assert oracle.within_tol(g32, y64, S, REL_TOL).all(), f"{label} vector {b} fp32 sums"


def oracle_sums(om, x):
    idx = np.nonzero(x != 0)[0].astype(np.int32)   # (NaN counts as active)
    ri, rv, rs = om.spmspv(idx, x[idx].astype(np.float64))
    y64, S = np.zeros(om.m), np.zeros(om.m)
    y64[ri], S[ri] = rv, rs
    return y64, S


def activations(nb, n, dtype, key, density=0.3):
    rng = wl.rng_for(wl.W_RAND, 120, key)
    X = np.where(rng.random((nb, n)) < density, rng.uniform(-1, 1, (nb, n)), 0.0).astype(dtype)
    X[0, : n // 3] = 0  # whole inactive vector blocks
    if nb > 2:
        X[1] = 0
    return X


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("force", [-1, 0, 1, 2, 3, 4])
def test_block_classes(torch, dtype, force):
    rng = wl.rng_for(wl.W_RAND, 121, force + 1)
    m, n = 90, 200
    # blocks from a few entries to full, column- and row-skewed ones among them
    p = np.kron(rng.choice([0.02, 0.1, 0.3, 0.6, 1.0], (6, 13)), np.ones((16, 16)))[:m, :n]
    keep = rng.random((m, n)) < p
    keep[16:32, 32:48] = False
    keep[16:32, [33, 40, 41]] = True          # column skew
    keep[32:48, 48:64] = False
    keep[[33, 40, 41], 48:64] = True          # row skew
    keep[48:64, 64:80] = False
    keep[50, 70] = True                       # one entry
    r, c = np.nonzero(keep)
    a = wl.csr_from_coo(m, n, r, c, wl._nonzero_uniform(rng, -1.0, 1.0, r.size, dtype=dtype))
    opts = dbs.default_opts(force_type=force, th1=250 if force == 4 else 128)
    A, om = gpu_matrix(a, opts), oracle_matrix(a)
    ctx = dbs.Context(A)
    for nb in (1, 2, 3, 8):
        check(ctx, A, om, activations(nb, n, dtype, nb), f"classes {dtype.__name__} force={force} nb={nb}")


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("m,n,keep", [(16, 2048, 0.5), (33, 4100, 0.4), (700, 3000, 0.1), (4096, 2100, 0.06),
                                      (17, 16, 0.5), (3290, 2064, 0.3), (32760, 250, 0.2), (32744, 250, 0.2),
                                      (32760, 16, 0.2), (40000, 33, 0.5)])
def test_shapes(torch, dtype, m, n, keep):
    """One block row in many parts, a few, the 16-wave shape (256 block rows),
    short rows, ragged both ways, many short rows (a wave each from 2048 on)."""
    rng = wl.rng_for(wl.W_RAND, 122, m, n)
    mask = rng.random((m, n)) < keep
    mask[16:32] &= n > 100                     # a block row without blocks in the narrow case
    r, c = np.nonzero(mask)
    a = wl.csr_from_coo(m, n, r, c, wl._nonzero_uniform(rng, -1.0, 1.0, r.size, dtype=dtype))
    A, om = gpu_matrix(a), oracle_matrix(a)
    ctx = dbs.Context(A)
    for nb in (1, 5):
        check(ctx, A, om, activations(nb, n, dtype, 10 + nb, 0.2), f"{dtype.__name__} {m}x{n} keep={keep} nb={nb}")


def layer(m, n, keep, dtype, key):
    """m x n, an entry with probability `keep`; block edges may be cut off."""
    rng = wl.rng_for(wl.W_RAND, 128, key)
    mask = rng.random((m, n)) < keep
    if m % 16 and n % 16:
        mask[m // 16 * 16:, n // 16 * 16:] = False  # (the corner block would be a COO block)
    r, c = np.nonzero(mask)
    return wl.csr_from_coo(m, n, r, c, wl._nonzero_uniform(rng, -1.0, 1.0, r.size, dtype=dtype))


@pytest.mark.parametrize("dtype,m,n,keep,nbs", [(np.float32, 6144, 2816, 0.4, (2,)), (np.float32, 4112, 4094, 0.4, (2, 3, 4)),
                                                (np.float32, 4112, 4094, 0.8, (2, 4)), (np.float32, 4100, 16, 0.85, (2, 3, 4)),
                                                (np.float16, 4100, 16, 0.85, (2,))])
def test_shared_lane_per_row_pass(torch, dtype, m, n, keep, nbs):
    """No COO block, 256 block rows and more: two fp32 vectors on 65536 blocks
    (four with 257 block rows), and up to four fp32 or two fp16 ones where block
    rows hold one block; and on either side of the rule the matrix cores, on the
    same context."""
    a = layer(m, n, keep, dtype, n)
    A, om = gpu_matrix(a), oracle_matrix(a)
    assert A.info()["blocks_by_type"]["coo"] == 0 and A.info()["nbr"] >= 256
    ctx = dbs.Context(A)
    for nb in (*nbs, max(nbs) + 1, 8, nbs[0]):
        check(ctx, A, om, activations(nb, n, dtype, 40 + nb), f"shared {dtype.__name__} {m}x{n} nb={nb}")


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("force", [1, 2, 3, 4])
def test_forced_formats_of_few_entries(torch, dtype, force):
    """Fewer than eight entries per block and no COO block: the lane-per-row
    pass for 2, 4 and 8 vectors."""
    a = layer(150, 330, 0.02, dtype, 500 + force)
    A, om = gpu_matrix(a, dbs.default_opts(force_type=force)), oracle_matrix(a)
    assert A.info()["nnz"] < 8 * A.info()["nblk"] and A.info()["blocks_by_type"]["coo"] == 0
    ctx = dbs.Context(A)
    for nb in (1, 2, 3, 4, 5, 8):
        check(ctx, A, om, activations(nb, 330, dtype, 50 + nb), f"few entries force={force} {dtype.__name__} nb={nb}")


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("th0", [32, 6])
def test_few_entries_with_coo_blocks(torch, dtype, th0):
    """Fewer than eight entries per block, COO blocks among them: one call per
    vector (th0 = 6: less than half of the entries in COO blocks)."""
    a = layer(150, 330, 0.025, dtype, 510)
    A, om = gpu_matrix(a, dbs.default_opts(th0=th0)), oracle_matrix(a)
    i = A.info()
    assert i["nnz"] < 8 * i["nblk"] and i["blocks_by_type"]["coo"] > 0
    ctx = dbs.Context(A)
    for nb in (1, 2, 5):
        check(ctx, A, om, activations(nb, 330, dtype, 60 + nb), f"few entries th0={th0} {dtype.__name__} nb={nb}")


@pytest.mark.parametrize("dtype,m,n,keep", [(np.float32, 2803, 5008, 0.95), (np.float32, 2003, 4499, 0.9),
                                            (np.float16, 2603, 6499, 0.95), (np.float32, 3000, 32, 0.3)])
def test_one_vector_beyond_the_matrix_core_pass(torch, dtype, m, n, keep):
    """One activation on layers that the matrix-core pass leaves to the scan
    and the traversal: more than 32 or 48 MiB of blocks, two blocks per block
    row; several vectors on them."""
    rng = wl.rng_for(wl.W_RAND, 129, m, n)
    mask = rng.random((m, n)) < keep
    mask[:16, :16] = False
    mask[3, 5] = True                      # (a COO block)
    r, c = np.nonzero(mask)
    a = wl.csr_from_coo(m, n, r, c, wl._nonzero_uniform(rng, -1.0, 1.0, r.size, dtype=dtype))
    A, om = gpu_matrix(a), oracle_matrix(a)
    ctx = dbs.Context(A)
    for nb in (1, 3):
        for density in (0.002, 0.3):
            check(ctx, A, om, activations(nb, n, dtype, 70 + nb, density), f"large {dtype.__name__} {m}x{n} nb={nb} {density}")


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_not_finite(torch, dtype):
    """Infinities and NaN reach the rows that hold the entry, and no others:
    not a row without the entry, not a token whose x is inactive there."""
    rng = wl.rng_for(wl.W_RAND, 123, 0)
    m, n = 70, 150
    r, c = np.nonzero(rng.random((m, n)) < 0.4)
    v = wl._nonzero_uniform(rng, -1.0, 1.0, r.size, dtype=dtype)
    a = wl.csr_from_coo(m, n, r, c, v)
    X = activations(4, n, dtype, 20, 0.5)
    X[2, 40:44] = [np.inf, 0.0, np.nan, -np.inf]
    for what in ("x", "A"):
        if what == "A":
            X = activations(4, n, dtype, 21, 0.5)
            a.vals[[5, 900, 2000]] = [np.inf, np.nan, -np.inf]
        A, om = gpu_matrix(a), oracle_matrix(a)
        ctx = dbs.Context(A)
        Y32 = torch.empty((4, m), dtype=torch.float32, device="cuda:0")
        ctx.spmm_dense(A, to_dev(X), Y32=Y32)
        torch.cuda.synchronize()
        for b in range(4):
            y64, _ = oracle_sums(om, X[b])
            g = Y32[b].cpu().numpy()
            log(f"not finite in {what}, vector {b}: {np.sum(~np.isfinite(y64))} rows")
            assert np.array_equal(np.isnan(g), np.isnan(y64))
            assert np.array_equal(np.isinf(g), np.isinf(y64)) and np.array_equal(g[np.isinf(g)], y64[np.isinf(y64)])
            ok = np.isfinite(y64)
            assert np.allclose(g[ok], y64[ok], rtol=0, atol=1e-5 * n)


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("force", [-1, 0, 1, 2, 3, 4])
def test_not_finite_in_long_block_rows(torch, dtype, force):
    """The second walk of a wave whose sums are not finite: every block class,
    more than 64 blocks per wave, a ragged last block, one block with an
    infinity and all of them."""
    rng = wl.rng_for(wl.W_RAND, 126, force + 1)
    m, n = 40, 5000
    p = np.kron(rng.choice([0.02, 0.1, 0.3, 0.6, 1.0], (3, 313)), np.ones((16, 16)))[:m, :n]
    r, c = np.nonzero(rng.random((m, n)) < p)
    a = wl.csr_from_coo(m, n, r, c, wl._nonzero_uniform(rng, -1.0, 1.0, r.size, dtype=dtype))
    opts = dbs.default_opts(force_type=force, th1=250 if force == 4 else 128)
    for case in ("x", "A", "last", "all of x"):
        X = activations(3, n, dtype, 30, 0.5)
        if case == "x":
            X[2, 4001] = np.inf
        elif case == "A":
            a.vals[[7, r.size // 2]] = [np.nan, -np.inf]
        elif case == "last":
            X[0, n - 1] = -np.inf
        else:
            X[:] = np.where(X > 0.5, np.inf, X)
        A, om = gpu_matrix(a, opts), oracle_matrix(a)
        Y32 = torch.empty((3, m), dtype=torch.float32, device="cuda:0")
        dbs.Context(A).spmm_dense(A, to_dev(X), Y32=Y32)
        torch.cuda.synchronize()
        for b in range(3):
            y64, S = oracle_sums(om, X[b])
            g = Y32[b].cpu().numpy()
            log(f"{case}, force={force} {dtype.__name__}, vector {b}: {np.sum(~np.isfinite(y64))} rows not finite")
            assert np.array_equal(np.isnan(g), np.isnan(y64))
            assert np.array_equal(g[np.isinf(y64)], y64[np.isinf(y64)]) and not np.isinf(g[np.isfinite(y64)]).any()
            ok = np.isfinite(y64)
            assert oracle.within_tol(g[ok], y64[ok], S[ok], REL_TOL).all()


def test_fp32_subnormals(torch):
    """Products and block sums below the smallest normal number are kept."""
    rng = wl.rng_for(wl.W_RAND, 127, 0)
    m, n = 64, 128
    r, c = np.nonzero(rng.random((m, n)) < 0.5)
    v = (rng.uniform(0.5, 1, r.size) * 1e-20).astype(np.float32)
    a = wl.csr_from_coo(m, n, r, c, v)
    X = np.where(rng.random((3, n)) < 0.5, rng.uniform(0.5, 1, (3, n)) * 1e-20, 0).astype(np.float32)
    A, om = gpu_matrix(a), oracle_matrix(a)
    Y = dbs.Context(A).spmm_dense(A, to_dev(X))
    torch.cuda.synchronize()
    for b in range(3):
        y64, _ = oracle_sums(om, X[b])
        # each of at most 128 products, and each block's sum, rounds by half of 2^-149
        d = np.abs(Y[b].cpu().numpy().astype(np.float64) - y64).max()
        log(f"fp32 subnormals, vector {b}: largest difference {d / 2.0 ** -149:.1f} of 2^-149, largest sum {y64.max():.2e}")
        assert d <= 140 * 2.0 ** -149


def test_fp16_subnormals(torch):
    rng = wl.rng_for(wl.W_RAND, 124, 0)
    m, n = 64, 128
    r, c = np.nonzero(rng.random((m, n)) < 0.5)
    v = (rng.integers(1, 1024, r.size) * 2.0 ** -24).astype(np.float16)      # subnormal weights
    a = wl.csr_from_coo(m, n, r, c, v)
    A, om = gpu_matrix(a), oracle_matrix(a)
    X = np.where(rng.random((3, n)) < 0.5, rng.uniform(1, 100, (3, n)), 0).astype(np.float16)
    X[1] = (rng.integers(0, 1024, n) * 2.0 ** -24).astype(np.float16)         # and a subnormal activation
    check(dbs.Context(A), A, om, X, "fp16 subnormals")


@pytest.mark.slow
@pytest.mark.parametrize("dtype,n", [(np.float32, 160_000_003), (np.float16, 310_000_000)])
def test_x_of_more_than_4_gib(torch, dtype, n):
    """Eight activations whose last one begins beyond 2^32 bytes of x."""
    rng = wl.rng_for(wl.W_RAND, 125, n)
    m, J = 20, np.array([0, 1, 777, n // 32, (n - 1) // 16 - 1, (n - 1) // 16], np.int64)
    assert 7 * n * np.dtype(dtype).itemsize > 1 << 32
    cols = (J[:, None] * 16 + np.arange(16)).reshape(-1)
    cols = cols[cols < n]
    W = np.where(rng.random((m, cols.size)) < 0.5, rng.uniform(0.1, 1, (m, cols.size)), 0).astype(dtype)
    X = rng.uniform(0.1, 1, (8, cols.size)).astype(dtype)
    X[:, ::3] = 0
    r, c = np.nonzero(W)
    A = gpu_matrix(wl.csr_from_coo(m, n, r, cols[c], W[r, c]))
    ctx = dbs.Context(A)
    x = torch.zeros((8, n), dtype=torch.float32 if dtype == np.float32 else torch.float16, device="cuda:0")
    x[:, torch.from_numpy(cols).cuda()] = to_dev(X)
    log(f"x of {x.numel() * x.element_size() >> 20} MiB, {dtype.__name__}")
    Y32 = torch.empty((8, m), dtype=torch.float32, device="cuda:0")
    ctx.spmm_dense(A, x, Y32=Y32)
    torch.cuda.synchronize()
    W64, X64 = W.astype(np.float64), X.astype(np.float64)
    ref, S = X64 @ W64.T, np.abs(X64) @ np.abs(W64).T
    for b in range(8):
        assert oracle.within_tol(Y32[b].cpu().numpy(), ref[b], S[b], REL_TOL).all(), f"vector {b}"
