"""The library's host side over a stand-in for the HIP runtime (fake_hip.py):
launch grids, allocation failures, which kernels a call takes."""
import fake_hip

# entries far apart: every block is a COO block of one entry, so that the
# matrix carries entry views
MATRIX = """
def list_matrix(m, n, per_row, dtype=np.float32):
    rp = np.arange(m + 1, dtype=np.int64) * per_row
    step = n // per_row
    ci = (np.arange(per_row)[None] * step + (np.arange(m)[:, None] * 17) % step).astype(np.int32)
    return m, n, rp, ci.reshape(-1), None if dtype is None else np.ones(m * per_row, dtype)

P = lambda a: None if a is None else ctypes.c_void_p(a.ctypes.data)

class Call:
    def __init__(self, *args, opts=None):
        self.A = dbs.Matrix.from_csr(*args, opts)
        self.ctx = ctypes.c_void_p()
        assert lib.dbs_ctx_create(self.A._h, None, ctypes.byref(self.ctx)) == 0, lib.dbs_last_error()
        m = self.A.m
        self.x, self.xv = np.arange(10, dtype=np.int32), np.ones(10, np.float32)
        self.y = np.zeros(m, np.int32), np.zeros(m, np.float32), np.zeros(1, np.int32)

    def pull(self):
        st = lib.dbs_spmspv(self.ctx, self.A._h, 0, 10, P(self.x), P(self.xv), None, 0, 2, 0.0, P(self.y[0]), P(self.y[1]),
                            P(self.y[2]), None)
        assert st == 0, lib.dbs_last_error()
        return fake.fake_grid()
"""


def test_grids_are_each_device_s_own():
    fake_hip.run(MATRIX + """
assert Call(*list_matrix(50000, 4000, 8)).pull() == 256
var("fake_device", ctypes.c_int).value = 1   # half of the compute units
assert Call(*list_matrix(50000, 4000, 8)).pull() == 128
var("fake_device", ctypes.c_int).value = 0
assert Call(*list_matrix(50000, 4000, 8)).pull() == 256
""")


def test_occupancy_is_not_asked_for_on_every_call():
    """Many matrices in turn, each with an LDS size of its own."""
    fake_hip.run(MATRIX + """
calls = [Call(*list_matrix(20, 2000 + 1000 * i, 8)) for i in range(40)]
for c in calls: c.pull()
asked = var("fake_occupancy_calls").value
assert asked >= 40
for c in calls: c.pull()
again = var("fake_occupancy_calls").value - asked
assert again <= 16, again    # (those that share a place in the table)
""")


def test_first_calls_from_many_threads():
    fake_hip.run(MATRIX + """
import threading
calls = [Call(*list_matrix(50000, 2000 + 1000 * (i % 12), 8)) for i in range(48)]
go, wrong = threading.Barrier(16), []
def work(t):
    go.wait()
    for i in range(t, 48, 16):
        for rep in range(3):
            g = calls[i].pull()
            if g != 256: wrong.append((i, g))
threads = [threading.Thread(target=work, args=(t,)) for t in range(16)]
for t in threads: t.start()
for t in threads: t.join()
assert not wrong, wrong
""")


ALLOCS = MATRIX + """
allocs, frees = var("fake_allocs"), var("fake_frees")
fail_at, fail_from = var("fake_fail_at"), var("fake_fail_from")

def failing(make, at=-1, frm=-1):
    '''(status, allocations, of them not freed) of make(out) with failures'''
    out = ctypes.c_void_p()
    allocs.value = frees.value = 0
    fail_at.value, fail_from.value = at, frm
    st = make(out)
    fail_at.value = fail_from.value = -1
    n = allocs.value
    failed = 0 if at < 0 and frm < 0 else 1 if at >= 0 and n > at else max(0, n - frm) if frm >= 0 else 0
    left = n - failed - frees.value
    if st == 0:
        lib.dbs_matrix_destroy(out)
        return st, n, n - failed - frees.value, left
    assert not out.value
    return st, n, left, left
"""


def test_upload_without_memory_for_the_views():
    """Every device allocation of an upload failing in turn: the entry views
    and the block list are left out, the format's own arrays are required;
    nothing leaks, and the matrix works."""
    fake_hip.run(ALLOCS + """
def upload(hm):
    return lambda out: lib.dbs_matrix_upload(hm._h, ctypes.byref(out))
host = lambda args, **o: dbs.HostMatrix.from_csr(*args, dbs.default_opts(**o))
rng = np.random.default_rng(1)
r, c = np.nonzero(rng.random((64, 64)) < 0.4)
filled = (64, 64, np.concatenate([[0], np.cumsum(np.bincount(r, minlength=64))]).astype(np.int64), c.astype(np.int32),
          np.ones(r.size, np.float32))
few = list_matrix(300, 300, 4)
_, base, _, _ = failing(upload(host(few, force_type=0)))      # (a forced format has no views)
for name, hm, more in (("views", host(few), True), ("pattern", host(list_matrix(300, 300, 4, None)), True),
                       ("list", host(filled), True), ("neither", host(few, force_type=0), False)):
    st, n, leak, kept = failing(upload(hm))
    assert st == 0 and leak == 0 and (n > base) == more, (name, n, base)
    for k in range(n):
        st, _, leak, kept = failing(upload(hm), at=k)
        assert leak == 0, (name, k, leak)
        assert (st == 0) == (k >= base), (name, k, base, st)
        if st == 0: assert kept < n, (name, k)
        st, _, leak, kept = failing(upload(hm), frm=k)
        assert leak == 0 and (st == 0) == (k >= base), (name, k, st)
# a matrix without views takes the scan and the block traversals: a launch more
full = Call(*few)
full.pull()
launches = var("fake_launches")
launches.value = 0; full.pull(); with_views = launches.value
fail_at.value = allocs.value + base
bare = Call(*few)
launches.value = 0; bare.pull()
assert launches.value > with_views, (launches.value, with_views)
""")


def test_conversion_without_memory_for_the_views():
    """Device allocations of dbs_matrix_build_dense: one that fails has it
    start once more without the optional arrays; none leaks."""
    fake_hip.run(ALLOCS + """
w = np.ones((100, 200), np.float32)
make = lambda out: lib.dbs_matrix_build_dense(100, 200, P(w), 200, 0, None, None, ctypes.byref(out))
st, n, leak, _ = failing(make)
assert st == 0 and leak == 0 and n > 10
for k in range(n):
    st, _, leak, _ = failing(make, at=k)
    assert st == 0 and leak == 0, (k, st, leak)
    st, _, leak, _ = failing(make, frm=k)
    assert st != 0 and leak == 0, (k, st, leak)
""")


def test_batch_scratch_that_could_not_be_had():
    """The second of the two batched buffers failing: the call reports it, the
    next one allocates both."""
    fake_hip.run(ALLOCS + """
rng = np.random.default_rng(2)
rows = np.repeat(np.arange(16), 2048)
cols = np.tile(np.arange(2048), 16)
rp = (np.arange(17) * 2048).astype(np.int64)
c = Call(16, 2048, rp, cols.astype(np.int32), np.ones(rows.size, np.float32))   # (a block row in parts)
x, y = np.ones((8, 2048), np.float32), np.zeros((8, 16), np.float32)
spmm = lambda: lib.dbs_spmm_dense(c.ctx, c.A._h, 8, P(x), P(y), None, None)
allocs.value = frees.value = 0
fail_at.value = 1
assert spmm() != 0
assert allocs.value == 2 and frees.value == 1
fail_at.value = -1
allocs.value = 0
assert spmm() == 0 and allocs.value == 2
allocs.value = 0
assert spmm() == 0 and allocs.value == 0
""")


ROUTES = MATRIX + """
import re
fake.fake_launched.restype = ctypes.c_char_p

def kernels(call):
    fake.fake_forget()
    assert call() == 0, lib.dbs_last_error()
    return re.findall("k_[a-z_]+[a-z]", fake.fake_launched().decode())

# nbr block rows of per_row blocks of 28 entries
def short_blocks(nbr, per_row, dtype=np.float32):
    cnt = np.tile(np.where(np.arange(16) < 14, 2 * per_row, 0), nbr)
    rp = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
    ci = np.tile((np.arange(per_row)[:, None] * 16 + np.arange(2)).reshape(-1), nbr * 14).astype(np.int32)
    return 16 * nbr, 16 * per_row, rp, ci, None if dtype is None else np.ones(ci.size, dtype)

def sparse(c, k, path, semiring=0):
    x, v = np.arange(k, dtype=np.int32), np.ones(k, np.float32)
    return kernels(lambda: lib.dbs_spmspv(c.ctx, c.A._h, semiring, k, P(x), P(v), None, 0, path, ctypes.c_float(0), P(c.y[0]),
                                          P(c.y[1]), P(c.y[2]), None))
"""


def test_pull_over_entries_or_blocks():
    """Sparse x: pull streams the entries up to a number of them, beyond it
    only with one or two per block; push walks the listed columns always."""
    fake_hip.run(ROUTES + """
AUTO, PUSH, PULL, OR_AND = 0, 1, 2, 1
for args, sr, stream in ((short_blocks(512, 640), 0, True), (short_blocks(1024, 640), 0, False),
                         (short_blocks(300, 640), OR_AND, True), (short_blocks(512, 640), OR_AND, False),
                         (short_blocks(512, 640, None), OR_AND, False), (list_matrix(1 << 20, 1 << 18, 16), 0, True),
                         (list_matrix(1 << 20, 1 << 18, 16), OR_AND, True)):
    c = Call(*args)
    few = c.A.n < 20000
    # (the last: a number of indices that does not settle the path)
    for k, path in ((50, PULL), (c.A.n // 2, AUTO), (40 if few else 2000, AUTO)):
        got = sparse(c, k, path, sr)
        assert ("k_entry_pull" in got) == stream and ("k_traverse" in got) == (not stream), (stream, k, path, got)
    got = sparse(c, 50, PUSH, sr)
    assert "k_entry_push" in got and "k_traverse" not in got, got
    del c
""", timeout=300)


def test_dense_activation_over_entries():
    """Short COO blocks: the stream alone up to 20M entries and for pull, beyond
    with the scan and the push kernel."""
    fake_hip.run(ROUTES + """
AUTO, PUSH, PULL = 0, 1, 2
for args, path, choose in ((short_blocks(512, 640), AUTO, False), (short_blocks(1200, 640), AUTO, True),
                           (short_blocks(1200, 640), PULL, False)):
    c = Call(*args)
    x, y = np.ones(c.A.n, np.float32), np.zeros(c.A.m, np.float32)
    got = kernels(lambda: lib.dbs_spmspv_dense(c.ctx, c.A._h, P(x), path, ctypes.c_float(0), P(y), None, None))
    assert "k_entry_pull" in got and ("k_scan" in got) == ("k_traverse" in got) == choose, (path, choose, got)
    del c
""", timeout=300)


def test_dense_activation_on_filled_blocks():
    """All blocks at once up to 32 MiB of them, 48 MiB with whole vector blocks,
    in either type; beyond the device chooses."""
    fake_hip.run(ROUTES + """
# blocks of 44 entries, the first one a COO block of 11; cut: the last vector block has 12 columns
def filled(nbr, nbc, dtype, cut):
    cols = np.add.outer(np.arange(nbc) * 16, np.arange(11)).reshape(-1).astype(np.int32)
    ci = np.concatenate([cols] + [cols[11:]] * 3 + [cols] * (4 * nbr - 4))
    cnt = np.tile(np.where(np.arange(16) < 4, cols.size, 0), nbr)
    cnt[1:4] -= 11
    return 16 * nbr, 16 * nbc - (4 if cut else 0), np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64), ci, np.ones(ci.size, dtype)

for dtype, nbr, cut, cores in ((np.float32, 480, False, True), (np.float32, 480, True, False), (np.float32, 600, False, False),
                               (np.float16, 800, False, True), (np.float16, 1000, False, False), (np.float16, 400, True, True)):
    c = Call(*filled(nbr, 450, dtype, cut))
    assert c.A.info()["blocks_by_type"]["coo"] == 1
    mib = (c.A.info()["nblk"] * 48 + c.A.info()["nnz"] * np.dtype(dtype).itemsize) / 2.0 ** 20
    assert (mib < (32 if cut else 48)) == cores, mib
    x, y = np.ones(c.A.n, dtype), np.zeros(c.A.m, dtype)
    got = kernels(lambda: lib.dbs_spmspv_dense(c.ctx, c.A._h, P(x), 0, ctypes.c_float(0), P(y), None, None))
    assert ("k_rows_mfma" in got) == cores and ("k_scan" in got) == (not cores), (dtype, nbr, cut, got)
    del c
""", timeout=300)


def test_batched_activations_on_uneven_block_rows():
    """fp32 layers without COO blocks: two vectors share the lane-per-row pass,
    up to four with 257 to 383 block rows (there of Dense blocks too if n is
    ragged); others take the matrix cores."""
    fake_hip.run(ROUTES + """
def layer(nbr, nbc, per, cut):   # per columns of every block row's blocks, in all 16 rows
    ci = np.tile(np.add.outer(np.arange(nbc) * 16, np.arange(per)).reshape(-1).astype(np.int32), 16 * nbr)
    return 16 * nbr, 16 * nbc - cut, (np.arange(16 * nbr + 1) * nbc * per).astype(np.int64), ci, np.ones(ci.size, np.float32)

for nbr, nbc, per, cut, most in ((256, 257, 4, 0, 2), (257, 256, 4, 0, 4), (383, 172, 4, 3, 4), (384, 172, 4, 0, 2), (257, 250, 4, 0, 0),
                                 (257, 256, 10, 0, 0), (257, 256, 10, 3, 4)):
    c = Call(*layer(nbr, nbc, per, cut))
    x, y = np.ones((5, c.A.n), np.float32), np.zeros((5, c.A.m), np.float32)
    for nb in (2, 3, 4, 5):
        got = kernels(lambda: lib.dbs_spmm_dense(c.ctx, c.A._h, nb, P(x), P(y), None, None))
        assert ("k_rows_mfma" in got) == (nb > most) and ("k_rows" in got) == (nb <= most), (nbr, nbc, per, cut, nb, got)
    del c
""", timeout=300)
