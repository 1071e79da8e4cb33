"""The library's host side over a stand-in for the HIP runtime (fake_hip.py):
launch grids, allocation failures."""
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
