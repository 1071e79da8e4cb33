"""GPU parity of BFS over the entry views (a kernel per level) against the
oracle: exact levels, parents and frontier sizes.

The graphs sit at the edges of its units: rows per wave (64, 256), entries a
lane looks at alone (1 + 8), the wave's rounds (64, then 512 and 4096 entries
of a row), levels launched ahead of the host (8), vertices that no edge leaves;
two hubs of more than 2^20 vertices put more found vertices into a workgroup
than its queue holds (1024 in pull, 4096 in push: emptied between turns)."""
import numpy as np
import pytest

import paper_2608_16308_amd as dbs
import workloads as wl
from gpu_helpers import gpu_matrix, log, oracle_matrix, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def graph(n, src, dst, symmetric=True):
    """Pattern with A[v][u] stored for every edge u -> v."""
    u, v = np.asarray(src, np.int64), np.asarray(dst, np.int64)
    key = np.unique(np.concatenate([v * n + u, u * n + v]) if symmetric else v * n + u)
    return wl.csr_from_coo(n, n, key // n, key % n)


def check(ctx, A, om, source, policy, th3, label):
    log(label)
    level, parent, st = ctx.bfs(A, source, policy=policy, th3=th3, stats=True)
    torch_mod().cuda.synchronize()
    el, ep, nl = om.bfs(source)
    assert np.array_equal(level.cpu().numpy(), el), f"{label}: levels"
    assert np.array_equal(parent.cpu().numpy(), ep), f"{label}: parents"
    assert st["levels"] == nl and st["reached"] == int((el >= 0).sum()), (label, st["levels"], nl)
    sizes = np.bincount(el[el >= 0], minlength=nl)[:64]
    assert st["frontier"] == sizes.tolist(), label


def graphs():
    rng = wl.rng_for(wl.W_RAND, 110, 0)
    yield "path 700", graph(700, np.arange(699), np.arange(1, 700))
    for n in (63, 64, 65, 255, 256, 257, 1025):
        yield f"random {n}", graph(n, rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n))
    # every vertex reached from one hub in one turn, and back
    n = 9000
    yield "star 9000", graph(n, np.full(n - 1, 4500), np.setdiff1d(np.arange(n), [4500]))
    # rows of 9, 10, 73, 74, 600 and 5000 entries whose only early column in
    # the frontier is the last one
    lens, n = [9, 10, 73, 74, 600, 5000], 12000
    src, dst = [0], [n - 1]
    for i, k in enumerate(lens):
        v = 100 + i
        src += list(200 + rng.choice(n - 300, k - 1, replace=False)) + [n - 1]
        dst += [v] * k
    yield "last column", graph(n, src, dst, symmetric=False)
    # 64 rows next to each other of 9,000 and more entries, a multiple of the
    # workgroup's 8192 and one more and less among them: reached in the first
    # or in the second step from the last vertex, or not at all; 32 of them are
    # read by the workgroup, the others by their wave
    n, late = 40000, 38000
    src, dst = [np.full(n - late - 1, n - 1)], [np.arange(late, n - 1)]
    for i in range(64):
        k = [9000, 584 + 8193, 584 + 16384, 585 + 16384, 583 + 24576, 30000][i % 6]
        cols = 200 + rng.choice(late - 1000, k - 1, replace=False)
        src.append(np.append(cols, late + i if i % 3 == 0 else late - 500 + i if i % 3 == 1 else 150))
        dst.append(np.full(k, 64 + i))
    hit = np.repeat(np.arange(late, n - 1), 30)   # the second step: the columns before `late`
    src.append(hit)
    dst.append(late - 700 + rng.integers(0, 700, hit.size))
    yield "long rows", graph(n, np.concatenate(src), np.concatenate(dst), symmetric=False)
    # directed, half of the vertices without outgoing edges
    n = 3000
    yield "dead ends", graph(n, rng.integers(0, n // 2, 9000), rng.integers(0, n, 9000), symmetric=False)
    yield "rmat15", wl.rmat(15, values=False)


@pytest.mark.parametrize("name", [name for name, _ in graphs()])
def test_bfs_over_entries(torch, name):
    a = next(g for k, g in graphs() if k == name)
    A, om = gpu_matrix(a), oracle_matrix(a)
    ctx = dbs.Context(A)
    for s in (0, a.n // 2, a.n - 1):
        for policy, th3 in (("auto", 0.0), ("push", 0.0), ("pull", 0.0), ("auto", 0.01), ("auto", 0.3)):
            check(ctx, A, om, s, policy, th3, f"{name} source={s} {policy} th3={th3}")


def test_bfs_wide_rows_per_turn(torch):
    """More than 2^20 vertices (256 rows per wave and turn), a ragged last
    turn, and a context that another, smaller graph uses in between."""
    n = (1 << 20) + 4099
    rng = wl.rng_for(wl.W_RAND, 111, 0)
    a = graph(n, rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n))
    b = graph(500, rng.integers(0, 500, 900), rng.integers(0, 500, 900))
    A, B, oa, ob = gpu_matrix(a), gpu_matrix(b), oracle_matrix(a), oracle_matrix(b)
    ctx = dbs.Context(A)
    for policy, th3 in (("auto", 0.0), ("pull", 0.0), ("auto", 0.05)):
        check(ctx, A, oa, n - 1, policy, th3, f"wide {policy} th3={th3}")
        check(ctx, B, ob, 7, policy, th3, f"small after wide {policy} th3={th3}")


def test_bfs_queues_overflow(torch):
    """A frontier of two hubs that finds 1.4M vertices: in push every workgroup
    takes about eight turns of 1024 entries and queues some 5,500 of the
    vertices, in pull more of them than its queue holds, so that the next
    level has no list (auto with th3: it is written from the bitmap)."""
    n = (1 << 20) + 500_003
    rng = wl.rng_for(wl.W_RAND, 112, 0)
    hub, other = n // 3, n // 2
    leaves = np.setdiff1d(np.arange(1, n), [hub, other])
    one, two = rng.random(leaves.size) < 0.7, rng.random(leaves.size) < 0.7
    a = graph(n, np.concatenate([[0, 0], np.full(one.sum(), hub), np.full(two.sum(), other)]),
              np.concatenate([[hub, other], leaves[one], leaves[two]]))
    A, om = gpu_matrix(a), oracle_matrix(a)
    ctx = dbs.Context(A)
    for s in (0, int(leaves[one & two][-1])):
        for policy, th3 in (("push", 0.0), ("pull", 0.0), ("auto", 0.0), ("auto", 0.01), ("auto", 2.0)):
            check(ctx, A, om, s, policy, th3, f"hubs source={s} {policy} th3={th3}")
