"""Timed cases of the library's public entry points, from the smallest calls
to the largest, over the kinds of matrix, vector and data type it serves.

``kind`` names the workload:

* ``uniform``  n x n, `per_row` distinct uniform columns per row, fp32; x of k
               uniform indices.  ``Context.spmspv_raw``.
* ``rmat``     power-law graph (R-MAT .57/.19/.19/.05, `edge_factor` generated
               edges per vertex, symmetrised, no self-loops, no duplicates,
               n need not be a power of two), fp32 values U(0,1); x uniform or
               in 64-aligned runs of 64.  ``Context.spmspv_raw``.
* ``mesh``     side^3 7-point stencil plus 5% uniform random entries, randomly
               relabelled, fp32 N(0,1); x the union of balls of 1024 grid
               points.  ``Context.spmspv_raw``.
* ``fem``      sx x sy x sz grid in natural order, 27-point stencil, 3 unknowns
               per node, fp32 N(0,1); x uniform.  ``Context.spmspv_raw``.
* ``or_and``   Boolean step on an R-MAT pattern with the complement of a
               visited set as output mask.  ``Context.spmspv_raw``.
* ``bfs``      a whole BFS, on an R-MAT pattern or on a FEM pattern.
* ``dense``    one dense activation (zeros skipped) against a pruned layer.
* ``batch``    several dense activations at once against a pruned layer.

Every input comes from the seed alone.  Outputs that have room for m entries
are zero behind the y_nnz entries a call writes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_16308_amd as dbs
from paper_2608_16308_amd import DBS_OR_AND

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a small sparse system, a handful of nonzeros in x: the cost of a call
        {"name": "uniform 4096, k=41", "kind": "uniform", "n": 4096, "per_row": 8, "k": 41},
        # graph propagation from a small, a middling and a large active set
        {"name": "rmat20 0.1% uniform", "kind": "rmat", "n": 1 << 20, "edge_factor": 16, "density": 0.001, "x": "uniform"},
        {"name": "rmat20 1% clustered", "kind": "rmat", "n": 1 << 20, "edge_factor": 16, "density": 0.01, "x": "clustered"},
        {"name": "rmat20 10% uniform", "kind": "rmat", "n": 1 << 20, "edge_factor": 16, "density": 0.1, "x": "uniform"},
        # a local update on a relabelled grid, sizes no multiple of anything
        {"name": "mesh 125^3 1% balls", "kind": "mesh", "side": 125, "density": 0.01},
        # a finite-element operator on a sparse load
        {"name": "fem 41^3x3 10%", "kind": "fem", "sx": 41, "sy": 41, "sz": 41, "density": 0.1},
        # one step of a user's own graph search, with its visited set as mask
        {"name": "or_and rmat18 masked", "kind": "or_and", "n": 1 << 18, "edge_factor": 16, "density": 0.02,
         "visited": 0.3},
        # BFS on a power-law graph (few large levels) and on a long FEM part
        # (many small ones)
        {"name": "bfs rmat22", "kind": "bfs", "graph": "rmat", "n": 1 << 22, "edge_factor": 16},
        {"name": "bfs fem 24x24x120x3", "kind": "bfs", "graph": "fem", "sx": 24, "sy": 24, "sz": 120},
        # decoding: one token and eight tokens through 50%-pruned fp16 layers
        {"name": "decode 11008x4096", "kind": "dense", "m": 11008, "n": 4096, "keep": 0.5, "active": 0.1, "dtype": "f16"},
        {"name": "decode 4096x14336 x8", "kind": "batch", "m": 4096, "n": 14336, "keep": 0.5, "active": 0.1,
         "dtype": "f16", "nb": 8},
        # a heavily pruned fp32 layer of odd sizes (its blocks are short lists)
        {"name": "pruned 95% 5003x7001 f32", "kind": "dense", "m": 5003, "n": 7001, "keep": 0.05, "active": 0.1,
         "dtype": "f32"},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["uniform", "rmat", "rmat", "mesh", "fem", "or_and", "bfs", "dense", "batch"])
    if kind == "uniform":
        n = _logint(rng, 1000, 60000)
        return {"kind": kind, "n": n, "per_row": rng.randint(4, 12), "k": max(1, int(n * math.exp(rng.uniform(-7, -2.5))))}
    if kind == "rmat":
        return {"kind": kind, "n": _logint(rng, 5000, 1 << 20), "edge_factor": rng.randint(6, 16),
                "density": round(10 ** rng.uniform(-4, -1), 6), "x": rng.choice(["uniform", "clustered"])}
    if kind == "mesh":
        return {"kind": kind, "side": _logint(rng, 17, 125), "density": round(10 ** rng.uniform(-3, -1), 5)}
    if kind == "fem":
        return {"kind": kind, "sx": rng.randint(5, 41), "sy": rng.randint(5, 41), "sz": rng.randint(5, 41),
                "density": round(10 ** rng.uniform(-3, -1), 5)}
    if kind == "or_and":
        return {"kind": kind, "n": _logint(rng, 4000, 1 << 19), "edge_factor": rng.randint(6, 16),
                "density": round(10 ** rng.uniform(-3, -1), 5), "visited": round(rng.uniform(0.0, 0.9), 3)}
    if kind == "bfs":
        if rng.random() < 0.5:
            return {"kind": kind, "graph": "rmat", "n": _logint(rng, 3000, 1 << 20), "edge_factor": rng.randint(6, 16)}
        return {"kind": kind, "graph": "fem", "sx": rng.randint(5, 24), "sy": rng.randint(5, 24), "sz": rng.randint(10, 120)}
    dtype = rng.choice(["f16", "f16", "f32"])
    keep = rng.choice([0.5, 0.5, 0.3, 0.05])
    m, n = _logint(rng, 600, 8000), _logint(rng, 600, 8000)
    if rng.random() < 0.5:
        m, n = (m + 15) // 16 * 16, (n + 15) // 16 * 16
    c = {"kind": kind, "m": m, "n": n, "keep": keep, "active": round(rng.uniform(0.03, 0.4), 3), "dtype": dtype}
    if kind == "batch":
        c["nb"] = rng.randint(2, 8)
    return c


# ---------------------------------------------------------------------------
# inputs (torch on the GPU, from the seed alone)
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream * 7919 + 12345) % (1 << 62))
    return g


def _rand(size, g, dtype=torch.float32):
    return torch.rand(size, generator=g, device=DEV, dtype=dtype)


def _values(size, g, normal):
    """fp32 values U(0,1) or N(0,1), none of them zero."""
    v = torch.randn(size, generator=g, device=DEV) if normal else _rand(size, g)
    return torch.where(v == 0, torch.full_like(v, 0.5), v)


def _csr(key, m, n):
    """(row_ptr int64, row int64, col int64) of sorted unique keys row * n + col."""
    row = torch.div(key, n, rounding_mode="floor")
    col = key - row * n
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(row, minlength=m), 0, out=row_ptr[1:])
    return row_ptr, row, col


def _rmat_keys(n, edge_factor, g):
    scale = max(1, (n - 1).bit_length())
    edges = n * edge_factor
    src = torch.zeros(edges, dtype=torch.int64, device=DEV)
    dst = torch.zeros(edges, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = _rand(edges, g)
        src = src * 2 + (r >= 0.76)
        dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    ok = (src != dst) & (src < n) & (dst < n)
    src, dst = src[ok], dst[ok]
    return torch.unique(torch.cat([src * n + dst, dst * n + src]))


def _fem_keys(sx, sy, sz, dof=3):
    nodes = sx * sy * sz
    v = torch.arange(nodes, dtype=torch.int64, device=DEV)
    x, y, z = v // (sy * sz), v // sz % sy, v % sz
    parts = []
    n = nodes * dof
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dz in (-1, 0, 1):
                ok = ((x + dx >= 0) & (x + dx < sx) & (y + dy >= 0) & (y + dy < sy) & (z + dz >= 0) & (z + dz < sz))
                a = v[ok]
                b = a + (dx * sy + dy) * sz + dz
                for p in range(dof):
                    for q in range(dof):
                        parts.append((a * dof + p) * n + b * dof + q)
    return torch.sort(torch.cat(parts)).values


def _grid_keys(side, g):
    n = side ** 3
    v = torch.arange(n, dtype=torch.int64, device=DEV)
    x, y, z = v // (side * side), v // side % side, v % side
    rows, cols = [v], [v]
    for coord, stride in ((x, side * side), (y, side), (z, 1)):
        for d in (-1, 1):
            ok = (coord + d >= 0) & (coord + d < side)
            rows.append(v[ok])
            cols.append(v[ok] + d * stride)
    r, c = torch.cat(rows), torch.cat(cols)
    extra = int(round(0.05 * r.numel()))
    er = torch.randint(0, n, (extra,), generator=g, device=DEV)
    ec = torch.randint(0, n, (extra,), generator=g, device=DEV)
    perm = torch.randperm(n, generator=g, device=DEV)
    return torch.unique(perm[torch.cat([r, er])] * n + perm[torch.cat([c, ec])]), perm


def _ball_x(side, k, perm, g):
    """k relabelled grid points in balls (by city-block distance) of 1024."""
    rad = 10
    o = torch.arange(-rad, rad + 1, device=DEV)
    dx, dy, dz = torch.meshgrid(o, o, o, indexing="ij")
    dist = (dx.abs() + dy.abs() + dz.abs()).reshape(-1)
    order = torch.sort(dist, stable=True).indices[:1024]
    off = torch.stack([dx.reshape(-1), dy.reshape(-1), dz.reshape(-1)], 1)[order]
    seeds = torch.randint(0, side, (max(1, -(-k // 1024) * 2), 3), generator=g, device=DEV)
    p = (seeds[:, None, :] + off[None]).reshape(-1, 3)
    p = p[((p >= 0) & (p < side)).all(1)]
    ids = (p[:, 0] * side + p[:, 1]) * side + p[:, 2]
    uniq, first = torch.unique(ids, return_inverse=True)
    seen = torch.full((uniq.numel(),), ids.numel(), dtype=torch.int64, device=DEV)
    seen.scatter_reduce_(0, first, torch.arange(ids.numel(), device=DEV), "amin")
    ids = uniq[torch.sort(seen).indices][:k]
    return torch.sort(perm[ids]).values


def _uniform_x(n, k, g):
    return torch.sort(torch.randperm(n, generator=g, device=DEV)[:k]).values


def _clustered_x(n, k, g):
    runs = min(-(-k // 64), n // 64)
    start = torch.randperm(n // 64, generator=g, device=DEV)[:runs] * 64
    idx = (start[:, None] + torch.arange(64, device=DEV)[None, :]).reshape(-1)[:k]
    return torch.sort(idx).values


def _activation(nb, n, active, g):
    """nb x n activations |N(0,1)|, round(active n) of each nonzero, 70% of
    those in a tenth of the 64-wide blocks."""
    k = max(1, int(round(active * n)))
    blocks = (n + 63) // 64
    hot = max(1, int(round(0.1 * blocks)))
    out = torch.zeros((nb, n), device=DEV)
    for b in range(nb):
        is_hot = torch.zeros(blocks, dtype=torch.bool, device=DEV)
        is_hot[torch.randperm(blocks, generator=g, device=DEV)[:hot]] = True
        h = is_hot.repeat_interleave(64)[:n]
        hp, cp = torch.nonzero(h).reshape(-1), torch.nonzero(~h).reshape(-1)
        kh = min(int(round(0.7 * k)), hp.numel())
        kc = min(k - kh, cp.numel())
        sel = torch.cat([hp[torch.randperm(hp.numel(), generator=g, device=DEV)[:kh]],
                         cp[torch.randperm(cp.numel(), generator=g, device=DEV)[:kc]]])
        out[b, sel] = _values(sel.numel(), g, True).abs().clamp(min=1e-4)
    return out


def _inputs(case, seed):
    """The case's matrix and vectors as torch tensors on the GPU."""
    kind, d = case["kind"], {}
    g, gx = _gen(seed, 1), _gen(seed, 2)
    if kind in ("dense", "batch"):
        m, n = case["m"], case["n"]
        dt = torch.float16 if case["dtype"] == "f16" else torch.float32
        w = torch.randn((m, n), generator=g, device=DEV) / math.sqrt(n)
        w = torch.where(w.abs() < 1e-6, torch.full_like(w, 1e-3), w)
        d["w"] = torch.where(_rand((m, n), g) < case["keep"], w, torch.zeros_like(w)).to(dt)
        d["a"] = _activation(case.get("nb", 1), n, case["active"], gx).to(dt)
        d["m"], d["n"] = m, n
        return d
    if kind == "uniform":
        n = case["n"]
        m = n
        r = torch.arange(n, device=DEV, dtype=torch.int64)[:, None]
        # distinct columns: a random start and distinct random steps per row
        lane = torch.arange(case["per_row"], device=DEV, dtype=torch.int64)
        c = torch.randint(0, n, (n, case["per_row"]), generator=g, device=DEV)
        c = (c // case["per_row"] * case["per_row"] + lane) % n
        key = torch.unique(r * n + c)
        d["idx"] = _uniform_x(n, case["k"], gx)
    elif kind in ("rmat", "or_and"):
        n = m = case["n"]
        key = _rmat_keys(n, case["edge_factor"], g)
        k = max(1, int(round(case["density"] * n)))
        d["idx"] = (_clustered_x if case.get("x") == "clustered" else _uniform_x)(n, k, gx)
        if kind == "or_and":
            bits = _rand((n + 31) // 32 * 32, gx) < case["visited"]
            bits[n:] = False
            sh = torch.arange(32, device=DEV, dtype=torch.int64)
            words = (bits.reshape(-1, 32).to(torch.int64) << sh).sum(1)
            d["mask"] = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
            d["visited"] = bits[:n]
    elif kind == "mesh":
        n = m = case["side"] ** 3
        key, perm = _grid_keys(case["side"], g)
        d["idx"] = _ball_x(case["side"], max(1, int(round(case["density"] * n))), perm, gx)
    elif kind == "fem" or case.get("graph") == "fem":
        n = m = case["sx"] * case["sy"] * case["sz"] * 3
        key = _fem_keys(case["sx"], case["sy"], case["sz"])
        if kind == "fem":
            d["idx"] = _uniform_x(n, max(1, int(round(case["density"] * n))), gx)
    else:
        n = m = case["n"]
        key = _rmat_keys(n, case["edge_factor"], g)
    d["m"], d["n"] = m, n
    d["row_ptr"], d["row"], d["col"] = _csr(key, m, n)
    if kind in ("uniform", "rmat", "mesh", "fem"):
        d["val"] = _values(key.numel(), g, kind in ("mesh", "fem"))
        d["xval"] = _values(d["idx"].numel(), gx, kind in ("mesh", "fem"))
    if kind == "bfs":
        deg = d["row_ptr"][1:] - d["row_ptr"][:-1]
        cand = torch.nonzero(deg >= min(3, int(deg.max()))).reshape(-1)
        d["source"] = int(cand[torch.randint(0, cand.numel(), (1,), generator=gx, device=DEV)])
    return d


# ---------------------------------------------------------------------------
# the entry points
# ---------------------------------------------------------------------------
def prepare(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    s = {"case": case}
    if kind in ("dense", "batch"):
        s["A"] = dbs.Matrix.from_dense(d["w"])
        s["x"] = d["a"] if kind == "batch" else d["a"][0].contiguous()
        s["y"] = torch.zeros((case["nb"], case["m"]) if kind == "batch" else (case["m"],), dtype=d["w"].dtype, device=DEV)
    else:
        val = d["val"].cpu().numpy() if "val" in d else None
        s["A"] = dbs.Matrix.from_csr(d["m"], d["n"], d["row_ptr"].cpu().numpy(), d["col"].to(torch.int32).cpu().numpy(), val)
        if "idx" in d:
            s["idx"] = d["idx"].to(torch.int32)
        s["xval"], s["mask"], s["source"] = d.get("xval"), d.get("mask"), d.get("source")
        if kind != "bfs":
            s["y_idx"] = torch.zeros(d["m"], dtype=torch.int32, device=DEV)
            s["y_val"] = None if kind == "or_and" else torch.zeros(d["m"], dtype=torch.float32, device=DEV)
            s["y_nnz"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        if kind == "bfs":
            s["level"] = torch.zeros(d["n"], dtype=torch.int32, device=DEV)
            s["parent"] = torch.zeros(d["n"], dtype=torch.int32, device=DEV)
    s["ctx"] = dbs.Context(s["A"])
    return s


def run(s):
    kind, A, ctx = s["case"]["kind"], s["A"], s["ctx"]
    if kind == "or_and":
        ctx.spmspv_raw(A, s["idx"], None, s["y_idx"], None, s["y_nnz"], semiring=DBS_OR_AND, mask=s["mask"],
                       complement=True)
        return s["y_idx"], s["y_nnz"]
    if kind == "bfs":
        return ctx.bfs(A, s["source"], level=s["level"], parent=s["parent"])
    if kind == "dense":
        return ctx.spmspv_dense(A, s["x"], y=s["y"])
    if kind == "batch":
        return ctx.spmm_dense(A, s["x"], Y=s["y"])
    ctx.spmspv_raw(A, s["idx"], s["xval"], s["y_idx"], s["y_val"], s["y_nnz"])
    return s["y_idx"], s["y_val"], s["y_nnz"]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what its outputs should be
# ---------------------------------------------------------------------------
def _nnz(case):
    kind = case["kind"]
    if kind == "uniform":
        return case["n"] * case["per_row"]
    if kind == "mesh":
        return 7.3 * case["side"] ** 3
    if "sx" in case:
        return 9.0 * (3 * case["sx"] - 2) * (3 * case["sy"] - 2) * (3 * case["sz"] - 2)
    return 1.87 * case["n"] * case["edge_factor"]


def work(case):
    """Sparse x: the stored entries of the columns x names (value and 4-byte
    position, 4 bytes for a pattern), x, and y (a row per entry, at most m).
    BFS: every stored entry's position once, level and parent.  Dense: the
    stored entries of the active columns (value and a byte of position)."""
    kind = case["kind"]
    if kind in ("dense", "batch"):
        nb, vb = case.get("nb", 1), 2 if case["dtype"] == "f16" else 4
        cols = 1.0 - (1.0 - case["active"]) ** nb
        nnz = case["m"] * case["n"] * case["keep"]
        return {"bytes": cols * nnz * (vb + 1) + nb * (case["m"] + case["n"]) * vb, "flops": 2 * case["active"] * nnz * nb}
    nnz = _nnz(case)
    m = case["side"] ** 3 if kind == "mesh" else 3 * case["sx"] * case["sy"] * case["sz"] if "sx" in case else case["n"]
    if kind == "bfs":
        return {"bytes": 4 * nnz + 8 * m, "flops": 0}
    density = case["k"] / case["n"] if kind == "uniform" else case["density"]
    useful = density * nnz
    if kind == "or_and":
        keep = 1 - case["visited"]
        return {"bytes": 4 * useful * keep + 4 * density * m + m / 8 + 4 * min(m, useful) * keep, "flops": useful * keep}
    return {"bytes": 8 * useful + 8 * density * m + 8 * min(m, useful), "flops": 2 * useful}


def tolerance(case):
    if case["kind"] in ("or_and", "bfs"):
        return "exact"
    if case.get("dtype") == "f16":
        # a sum near the middle of two fp16 numbers may round to either (2e-4
        # off the fp64 sums, all of it the rounding to fp16)
        return {"rel": 1e-4, "max": 2e-3}
    # fp32 products and one rounding of the sum: 3e-8 to 6e-8 off fp64
    return {"rel": 3e-7, "max": 6e-6}


def _spmspv64(d, m):
    """(rows with a product, ascending; their fp64 sums or None)"""
    x = torch.zeros(d["n"], dtype=torch.float64, device=DEV)
    on = torch.zeros(d["n"], dtype=torch.bool, device=DEV)
    on[d["idx"]] = True
    hit = on[d["col"]]
    row, col = d["row"][hit], d["col"][hit]
    if "val" not in d:
        return torch.unique(row), None
    x[d["idx"]] = d["xval"].double()
    y = torch.zeros(m, dtype=torch.float64, device=DEV)
    y.index_add_(0, row, d["val"][hit].double() * x[col])
    rows = torch.unique(row)
    return rows, y[rows]


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("dense", "batch"):
        y = torch.stack([d["w"].double() @ a.double() for a in d["a"]])
        return y if kind == "batch" else y[0]
    m = d["m"]
    if kind == "bfs":
        level = torch.full((m,), -1, dtype=torch.int32, device=DEV)
        parent = torch.full((m,), -1, dtype=torch.int64, device=DEV)
        front = torch.tensor([d["source"]], device=DEV)
        level[front], parent[front] = 0, d["source"]
        depth = 0
        while front.numel():
            on = torch.zeros(m, dtype=torch.bool, device=DEV)
            on[front] = True
            e = on[d["col"]] & (level[d["row"]] < 0)
            row, col = d["row"][e], d["col"][e]
            low = torch.full((m,), m, dtype=torch.int64, device=DEV)
            low.scatter_reduce_(0, row, col, "amin")
            front = torch.nonzero(low < m).reshape(-1)
            depth += 1
            level[front], parent[front] = depth, low[front]
        return level, parent.to(torch.int32)
    rows, val = _spmspv64(d, m)
    if kind == "or_and":
        rows = rows[~d["visited"][rows]]
    k = rows.numel()
    y_nnz = torch.tensor([k], dtype=torch.int32, device=DEV)
    y_idx = torch.zeros(m, dtype=torch.int32, device=DEV)
    y_idx[:k] = rows.to(torch.int32)
    if kind == "or_and":
        return y_idx, y_nnz
    y_val = torch.zeros(m, dtype=torch.float64, device=DEV)
    y_val[:k] = val
    return y_idx, y_val, y_nnz
