// gfx950 BFS over the entry views (Sec. 4.2, Alg. 5): a level is one kernel,
// and levels are launched without waiting for the host.
//
// The frontier of level l is a bitmap and, for push, a list of work items;
// V holds the vertices of the levels before it, so that "reached" during
// level l is V | F, which nothing in the level changes (V |= F, done by the
// same kernel, leaves it as it is).  Three bitmaps and three count records
// take turns as this level's, the next level's and the one being cleared.
//
//   push (top-down): the entries of the frontier's columns, 64 per wave step;
//     an unreached row takes the smallest frontier column by an atomic
//     minimum on its parent, and whoever finds the parent unset owns the row:
//     it writes the level, the next bitmap and the next work item.
//   pull (bottom-up): every unreached row looks for its first column in the
//     frontier, in ascending order, and stops there: that column is its
//     smallest-id parent.  The first column of each row sits in the row
//     table, so that most rows (on R-MAT 20: 61-99% of those found) are
//     settled without reading their entries; then a lane takes up to eight
//     more entries, then the wave.
//
// A segment-wise pull has to visit every block of a block row with an
// unreached row: on R-MAT 22 (128M entries) the largest level took 580-820 us
// that way, mostly one mask gather per block.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"
#include "turn_queue.hpp"

namespace dbs {

constexpr int BL_TPB = 1024;
constexpr int BL_WAVES = BL_TPB / WAVE;
constexpr int BL_PUSH_QUEUE = 4096;  // found vertices queued in LDS before their items are written
constexpr int BL_PULL_QUEUE = 1024;  // pull: with more per workgroup the next level pulls again
constexpr int BL_ROWS = 256;         // rows per wave and turn of pull, at most
constexpr int BL_LANE = 8;           // entries a lane looks at alone
// Rows with more than BL_LONG entries left after a wave's first two rounds
// (584 entries) are read by the whole workgroup, up to BL_LONG_ROWS of them: a
// row of 2^20 entries without a parent in the frontier took its wave 9 ms a
// level (a BFS that meets four of them in three levels 110 ms, with the
// workgroup 4.3; R-MAT and stencils, which have few such rows, within 1%).
constexpr int32_t BL_LONG = 8192;
constexpr int BL_LONG_ROWS = 32;

struct BfsArgs {
    const int2 *rowinfo;
    const uint32_t *col;
    const int32_t *row, *chord;
    int32_t nchunk;
    int32_t stream;     // a forced path or an explicit th3: sparse pull levels stream
    const int32_t *ce_ptr, *ce_row;
    int32_t n, nwords;
    uint32_t *vis;
    uint32_t *bits[3];
    int4 *items[2];
    BfsCount *cnt;
    BfsRecord *rec;
    int32_t *level;
    uint32_t *parent;   // (-1 is the largest unsigned value)
    int32_t policy;     // 0 auto, else PATH_PUSH / PATH_PULL
    double th3n;        // > 0: push iff nonzero vector blocks < th3n
    int64_t nnz;
    int64_t push_max;   // else the entries of a frontier that pushes whatever the rest, if it is listed (k_bfs_level)
};

struct BfsLds {
    union {
        struct {  // found vertices: id, first column entry, number of them
            int32_t v[BL_PUSH_QUEUE], p[BL_PUSH_QUEUE], len[BL_PUSH_QUEUE];
        } q;
        struct {
            int32_t q[BL_PULL_QUEUE];
            // rows a wave has not settled from the row table
            uint16_t row[BL_WAVES][BL_ROWS];
            int32_t beg[BL_WAVES][BL_ROWS], end[BL_WAVES][BL_ROWS];
            uint32_t out[BL_WAVES][BL_ROWS / 32];  // rows found
            uint32_t hit[BL_WAVES][WAVE];          // column found for a lane's row
            // long rows: id, next entry, end, entries for the count of those found
            int32_t lv[BL_LONG_ROWS], lp[BL_LONG_ROWS], le[BL_LONG_ROWS], ln[BL_LONG_ROWS];
        } pull;
    };
    uint64_t tot[BL_WAVES];
    uint64_t base, ent;
    uint32_t nq, found, inc, nvb;
    uint32_t nlong, lhit;
};

// The push queue of a workgroup (queue_is_full).
struct BfsQueueOps {
    BfsLds &L;
    __device__ __forceinline__ void barrier() { __syncthreads(); }
    __device__ __forceinline__ uint32_t count() { return L.nq; }
};

__device__ __forceinline__ bool bit_of(const uint32_t *b, uint32_t i) { return (b[i >> 5] >> (i & 31)) & 1u; }

// Writes the items of n found vertices (id, first column entry and count by
// at(i); vertices without column entries get none and are only counted).
// Called by the whole workgroup, after a barrier.
template <class At>
__device__ __forceinline__ void bfs_flush(BfsLds &L, BfsCount *next, int4 *items, int32_t n, At &&at)
{
    const int t = threadIdx.x, lane = lane_id(), wv = wave_id();
    for (int32_t i0 = 0; i0 < n; i0 += BL_TPB) {
        const bool on = i0 + t < n;
        int32_t v = 0, p = 0, len = 0;
        if (on) at(i0 + t, v, p, len);
        const uint64_t mine = len > 0 ? (1ull << EV_TASK_BITS) + (uint64_t)len : 0ull;
        const uint64_t none = ballot(on && len == 0);
        if (lane == 0 && none) atomicAdd(&next->extra, (uint32_t)__popcll(none));
        uint64_t inc = mine;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const uint64_t u = (uint64_t)__shfl_up((unsigned long long)inc, o, WAVE);
            if (lane >= o) inc += u;
        }
        if (lane == WAVE - 1) L.tot[wv] = inc;
        __syncthreads();
        if (t == 0) {
            uint64_t tot = 0;
#pragma unroll
            for (int i = 0; i < BL_WAVES; ++i) {
                const uint64_t u = L.tot[i];
                L.tot[i] = tot;
                tot += u;
            }
            L.base = tot ? (uint64_t)atomicAdd((unsigned long long *)&next->items, (unsigned long long)tot) : 0ull;
        }
        __syncthreads();
        if (mine) {
            const uint64_t to = L.base + L.tot[wv] + inc - mine;
            const int32_t first = (int32_t)(to & ((1ull << EV_TASK_BITS) - 1));
            items[to >> EV_TASK_BITS] = make_int4(first, p - first, v, 0);
        }
        __syncthreads();
    }
}

// Whether a pull level streams the entries (k_bfs_stream).
__device__ __forceinline__ bool bfs_stream(const BfsArgs &a, const BfsCount &c)
{
    const int64_t mf = (int64_t)(c.items & ((1ull << EV_TASK_BITS) - 1)) + (int64_t)c.ent;
    return a.stream && mf * 64 < a.nnz;
}

// Four consecutive column words from a 4-byte aligned place.
struct __attribute__((packed, aligned(4))) Cols4 {
    uint32_t c[4];
};

// G: rows per wave and turn of pull, in waves of 64 -- four where that leaves
// every wave a turn (their table loads are in flight together), else one.
template <int G>
__global__ __launch_bounds__(BL_TPB, 8) void k_bfs_level(BfsArgs a, int32_t l)
{
    __shared__ BfsLds L;
    const int t = threadIdx.x, lane = lane_id(), wv = wave_id();
    const BfsCount c = a.cnt[l % 3];
    const uint32_t *F = a.bits[l % 3];
    uint32_t *nb = a.bits[(l + 1) % 3], *clr = a.bits[(l + 2) % 3];
    const int32_t gt = blockIdx.x * BL_TPB + t;
    const uint32_t f0 = gt < a.nwords ? F[gt] : 0u;  // (for V |= F below)
    BfsCount *next = &a.cnt[(l + 1) % 3];
    const uint32_t NT = (uint32_t)(c.items >> EV_TASK_BITS), found = NT + c.extra;
    const int64_t T = (int64_t)(c.items & ((1ull << EV_TASK_BITS) - 1));
    const bool lead = blockIdx.x == 0 && t == 0;
    if (lead) a.cnt[(l + 2) % 3] = BfsCount{};
    if (found == 0) return;  // the BFS has ended
    // The automatic rule was found on R-MAT 22 and a stencil of 207,360 rows
    // (a push of under 2% of the entries only: the stencil's fronts then pull,
    // and every row not reached is read to its end, 185 us a level; the growth
    // bound keeps the power law's exploding levels at pull).
    const int64_t mf = T + (int64_t)c.ent;             // entries of the frontier
    const int64_t mu = a.nnz - (int64_t)c.seen - mf;   // and of the vertices not reached
    const bool push =
        a.policy == PATH_PUSH ||
        (a.policy == 0 && (a.th3n > 0.0 ? (double)c.nvb < a.th3n
                                        : !c.inc && (mf < a.push_max ||
                                                     (mf < mu && mf < 5 * a.push_max && mf < 4 * (int64_t)c.prev))));
    if (lead) {
        next->seen = c.seen + (uint64_t)mf;
        next->prev = (uint64_t)mf;
        a.rec->levels = l + 1;
        a.rec->reached += (int32_t)found;
        if (l < BFS_RECORD_LEVELS) {
            a.rec->path[l] = push ? PATH_PUSH : PATH_PULL;
            a.rec->frontier[l] = (int32_t)found;
        }
    }
    int4 *const nitems = a.items[(l + 1) & 1];
    const bool nvb = a.th3n > 0.0;
    if (t == 0) {
        L.nq = L.found = L.inc = L.nvb = L.nlong = 0;
        L.lhit = 0xFFFFFFFFu;
        L.ent = 0;
    }
    __syncthreads();
    if (push) {
        const int4 *items = a.items[l & 1];
        auto flush = [&](uint32_t n) {
            bfs_flush(L, next, nitems, (int32_t)n, [&](int32_t i, int32_t &v, int32_t &p, int32_t &len) {
                v = L.q.v[i];
                p = L.q.p[i];
                len = L.q.len[i];
            });
        };
        BfsQueueOps ops{L};
        uint32_t room = BL_PUSH_QUEUE, queued = 0;
        for (int64_t u0 = (int64_t)blockIdx.x * BL_WAVES; u0 * WAVE < T; u0 += (int64_t)gridDim.x * BL_WAVES) {
            if (queue_is_full<BL_PUSH_QUEUE, BL_TPB>(room, queued, ops)) {
                flush(queued);
                if (t == 0) L.nq = 0;
                __syncthreads();
            }
            const int64_t tb = (u0 + wv) * WAVE;
            if (tb < T) {
                const int32_t t0 = (int32_t)tb, tt = t0 + lane;
                int32_t lo = 0, hi = (int32_t)NT;
                while (hi - lo > 1) {
                    const int32_t step = (hi - lo + WAVE - 1) / WAVE, pi = lo + lane * step;
                    const int32_t x = pi < hi ? items[pi].x : INT_MAX;
                    const int q = 63 - __builtin_clzll(ballot(x <= t0));  // lane 0 probes lo: always set
                    lo += q * step;
                    hi = min(hi, lo + step);
                }
                const int4 it = lo + lane < (int32_t)NT ? items[lo + lane] : make_int4(INT_MAX, 0, 0, 0);
                int s = 0;
#pragma unroll
                for (int st = 32; st > 0; st >>= 1) {
                    const int32_t x = __shfl(it.x, s + st, WAVE);
                    if (s + st < WAVE && x <= tt) s += st;
                }
                const int32_t e = __shfl(it.y, s, WAVE) + tt;
                const uint32_t from = (uint32_t)__shfl(it.z, s, WAVE);
                bool first = false;
                int32_t v = 0, p = 0, len = 0;
                if (tt < T) {
                    v = a.ce_row[e];
                    const uint32_t seen = a.vis[v >> 5] | F[v >> 5];
                    if (!((seen >> (v & 31)) & 1u)) {
                        // (the column's extent goes out with the atomic)
                        p = a.ce_ptr[v];
                        len = a.ce_ptr[v + 1] - p;
                        first = atomicMin(&a.parent[v], from) == 0xFFFFFFFFu;
                    }
                }
                if (first) {
                    a.level[v] = l + 1;
                    const uint32_t bit = 1u << (v & 31);
                    if (nvb) {
                        if (!((atomicOr(&nb[v >> 5], bit) >> (v & 16)) & 0xFFFFu)) atomicAdd(&L.nvb, 1u);
                    } else {
                        atomicOr(&nb[v >> 5], bit);
                    }
                }
                const uint64_t m = ballot(first);
                if (m) {
                    uint32_t at = 0;
                    if (lane == 0) at = atomicAdd(&L.nq, (uint32_t)__popcll(m));
                    at = readlane_u32(at, 0) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    if (first) {
                        L.q.v[at] = v;
                        L.q.p[at] = p;
                        L.q.len[at] = len;
                    }
                }
            }
        }
        if (gt < a.nwords) {
            if (f0) a.vis[gt] |= f0;
            clr[gt] = 0u;
        }
        __syncthreads();  // (nothing is queued after it)
        if (L.nq) flush(L.nq);
    } else if (bfs_stream(a, c)) {  // (k_bfs_stream has found the level)
        if (gt < a.nwords) {
            if (f0) a.vis[gt] |= f0;
            clr[gt] = 0u;
        }
    } else {
        constexpr int ROWS = G * WAVE;
        // a wave takes ROWS consecutive rows per turn; no wave waits for
        // another until the end
        const int32_t nturn = (a.n + ROWS - 1) / ROWS;
        uint16_t *lrow = L.pull.row[wv];
        int32_t *lbeg = L.pull.beg[wv], *lend = L.pull.end[wv];
        uint32_t *out = L.pull.out[wv];
        const uint64_t below = (1ull << lane) - 1ull;
        int64_t ents = 0;  // entries of the rows this lane found
        for (int32_t turn = wv * (int32_t)gridDim.x + (int32_t)blockIdx.x; turn < nturn;
             turn += (int32_t)gridDim.x * BL_WAVES) {
            const int32_t v0 = turn * ROWS, w0 = v0 >> 5;
            uint32_t seen = 0xFFFFFFFFu;
            if (lane < ROWS / 32 && w0 + lane < a.nwords) seen = a.vis[w0 + lane] | F[w0 + lane];
            if (!ballot(seen != 0xFFFFFFFFu)) continue;
            // the row table of all unreached rows, then their first columns
            int2 ri[G];
            int32_t en[G];
            bool un[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int32_t v = v0 + g * WAVE + lane;
                const uint32_t w = (uint32_t)__shfl((int)seen, g * 2 + (lane >> 5), WAVE);
                un[g] = v < a.n && !((w >> (lane & 31)) & 1u);
                ri[g] = un[g] ? a.rowinfo[v] : make_int2(0, 0);
                en[g] = un[g] ? a.rowinfo[v + 1].x : 0;
            }
            uint32_t fw[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                un[g] = un[g] && ri[g].x < en[g];
                fw[g] = un[g] ? F[(uint32_t)ri[g].y >> 5] : 0u;
            }
            uint32_t nl = 0, cnt = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int32_t v = v0 + g * WAVE + lane;
                const bool hit = (fw[g] >> (ri[g].y & 31)) & 1u;
                if (hit) {
                    a.parent[v] = (uint32_t)ri[g].y;
                    a.level[v] = l + 1;
                    ents += en[g] - ri[g].x;
                }
                const uint64_t m = ballot(hit);
                cnt += (uint32_t)__popcll(m);
                if (lane < 2) out[g * 2 + lane] = (uint32_t)(m >> (32 * lane));
                const bool open = un[g] && !hit && ri[g].x + 1 < en[g];
                const uint64_t o = ballot(open);
                if (open) {
                    const uint32_t at = nl + (uint32_t)__popcll(o & below);
                    lrow[at] = (uint16_t)(g * WAVE + lane);
                    lbeg[at] = ri[g].x + 1;
                    lend[at] = en[g];
                }
                nl += (uint32_t)__popcll(o);
            }
            wave_lds_sync();
            // the open rows, a lane each
            for (uint32_t i0 = 0; i0 < nl; i0 += WAVE) {
                const bool on = i0 + lane < nl;
                const int32_t r = on ? lrow[i0 + lane] : 0, end = on ? lend[i0 + lane] : 0;
                const int32_t beg = on ? lbeg[i0 + lane] : 0;
                int32_t p = beg;
                uint32_t hit = 0xFFFFFFFFu;
                if (on) {
                    // (the array is padded: the words past the row are not used)
                    const Cols4 ca = *(const Cols4 *)(a.col + p), cb = *(const Cols4 *)(a.col + p + 4);
                    uint32_t cw[BL_LANE], f[BL_LANE];
#pragma unroll
                    for (int k = 0; k < BL_LANE; ++k) cw[k] = (k < 4 ? ca.c[k & 3] : cb.c[k & 3]) & ~RE_START;
#pragma unroll
                    for (int k = 0; k < BL_LANE; ++k) f[k] = p + k < end ? F[cw[k] >> 5] : 0u;
#pragma unroll
                    for (int k = BL_LANE - 1; k >= 0; --k)
                        if ((f[k] >> (cw[k] & 31)) & 1u) hit = cw[k];
                }
                p += BL_LANE;
                // rows still open: the wave takes up to `most` further entries
                // of each, numbered through, then looks which rows remain
                bool open = on && hit == 0xFFFFFFFFu && p < end;
                uint32_t *hl = L.pull.hit[wv];
                for (int32_t most = WAVE; ballot(open); most = min(most * 8, 4096)) {
                    const int32_t take = open ? min(end - p, most) : 0;
                    const int32_t inc = (int32_t)wave_incl_add((uint32_t)take), exc = inc - take;
                    const int32_t tot = (int32_t)readlane_u32((uint32_t)inc, WAVE - 1);
                    hl[lane] = 0xFFFFFFFFu;
                    wave_lds_sync();
                    auto step = [&](int32_t g0, auto U) {
                        constexpr int N = decltype(U)::value;
                        uint32_t cw[N], f[N];
                        int s[N];
#pragma unroll
                        for (int k = 0; k < N; ++k) {
                            // the last row that starts at or before entry g
                            // (rows without a share start where the next does)
                            const int32_t g = g0 + k * WAVE + lane;
                            s[k] = 0;
#pragma unroll
                            for (int st = 32; st > 0; st >>= 1) {
                                const int32_t x = __shfl(exc, s[k] + st, WAVE);
                                if (s[k] + st < WAVE && x <= g) s[k] += st;
                            }
                            const int32_t e = __shfl(p, s[k], WAVE) + g - __shfl(exc, s[k], WAVE);
                            cw[k] = g < tot ? a.col[e] & ~RE_START : 0u;
                        }
#pragma unroll
                        for (int k = 0; k < N; ++k) f[k] = g0 + k * WAVE + lane < tot ? F[cw[k] >> 5] : 0u;
#pragma unroll
                        for (int k = 0; k < N; ++k)
                            if ((f[k] >> (cw[k] & 31)) & 1u) atomicMin(&hl[s[k]], cw[k]);
                    };
                    int32_t g0 = 0;
                    for (; g0 + 8 * WAVE <= tot; g0 += 8 * WAVE) step(g0, std::integral_constant<int, 8>{});
                    for (; g0 < tot; g0 += 2 * WAVE) step(g0, std::integral_constant<int, 2>{});
                    wave_lds_sync();
                    const uint32_t got = hl[lane];
                    wave_lds_sync();
                    p += take;
                    if (open) hit = got;
                    open = open && got == 0xFFFFFFFFu && p < end;
                    if (most > WAVE && open && end - p > BL_LONG) {
                        const uint32_t at = atomicAdd(&L.nlong, 1u);
                        if (at < BL_LONG_ROWS) {
                            L.pull.lv[at] = v0 + r;
                            L.pull.lp[at] = p;
                            L.pull.le[at] = end;
                            L.pull.ln[at] = end - beg;
                            open = false;
                        }
                    }
                }
                const bool h = hit != 0xFFFFFFFFu;
                if (h) {
                    a.parent[v0 + r] = hit;
                    a.level[v0 + r] = l + 1;
                    ents += end - beg;
                    atomicOr(&out[r >> 5], 1u << (r & 31));
                }
                cnt += (uint32_t)__popcll(ballot(h));
            }
            if (!cnt) continue;
            wave_lds_sync();
            const uint32_t ow = lane < ROWS / 32 ? out[lane] : 0u;
            if (ow) nb[w0 + lane] = ow;
            if (nvb) {
                const uint32_t k = wave_sum(((ow & 0xFFFFu) ? 1u : 0u) + ((ow >> 16) ? 1u : 0u));
                if (lane == 0) atomicAdd(&L.nvb, k);
            }
            uint32_t at = 0;
            if (lane == 0) {
                atomicAdd(&L.found, cnt);
                at = atomicAdd(&L.nq, cnt);
            }
            at = readlane_u32(at, 0);
            if (at + cnt > BL_PULL_QUEUE) {
                if (lane == 0) L.inc = 1u;  // too many for push items
            } else {
                const uint32_t inc = wave_incl_add(__popc(ow));
                uint32_t w = ow, to = at + inc - __popc(ow);
                while (w) {
                    L.pull.q[to++] = v0 + lane * 32 + ctz32(w);
                    w &= w - 1u;
                }
            }
            wave_lds_sync();
        }
        if (gt < a.nwords) {
            if (f0) a.vis[gt] |= f0;
            clr[gt] = 0u;
        }
        ents = wave_sum(ents);
        if (lane == 0 && ents) atomicAdd((unsigned long long *)&L.ent, (unsigned long long)ents);
        __syncthreads();
        const uint32_t nlong = min(L.nlong, (uint32_t)BL_LONG_ROWS);  // (nothing is added after the barrier)
        if (nlong) {
            // (the words of the next bitmap that other waves stored are in memory)
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        for (uint32_t i = 0; i < nlong; ++i) {
            const int32_t end = L.pull.le[i];
            uint32_t got = 0xFFFFFFFFu;
            for (int64_t p = L.pull.lp[i]; p < end && got == 0xFFFFFFFFu; p += BL_LANE * BL_TPB) {
                const int32_t left = end - (int32_t)p;
                uint32_t cw[BL_LANE], f[BL_LANE], hit = 0xFFFFFFFFu;
#pragma unroll
                for (int k = 0; k < BL_LANE; ++k) cw[k] = k * BL_TPB + t < left ? a.col[p + k * BL_TPB + t] & ~RE_START : 0u;
#pragma unroll
                for (int k = 0; k < BL_LANE; ++k) f[k] = k * BL_TPB + t < left ? F[cw[k] >> 5] : 0u;
#pragma unroll
                for (int k = BL_LANE - 1; k >= 0; --k)
                    if ((f[k] >> (cw[k] & 31)) & 1u) hit = cw[k];
                if (hit != 0xFFFFFFFFu) atomicMin(&L.lhit, hit);
                __syncthreads();
                got = L.lhit;
                __syncthreads();  // (no thread is at the next entries before every thread has read it)
            }
            if (got == 0xFFFFFFFFu) continue;
            if (t == 0) {
                const int32_t v = L.pull.lv[i];
                a.parent[v] = got;
                a.level[v] = l + 1;
                const uint32_t old = atomicOr(&nb[v >> 5], 1u << (v & 31));
                if (!((old >> (v & 16)) & 0xFFFFu)) ++L.nvb;
                ++L.found;
                L.ent += (uint64_t)L.pull.ln[i];
                const uint32_t at = L.nq++;
                if (at < BL_PULL_QUEUE) L.pull.q[at] = v;
                else L.inc = 1u;
                L.lhit = 0xFFFFFFFFu;
            }
            __syncthreads();
        }
        if (L.inc) {
            if (t == 0) {
                atomicAdd(&next->extra, L.found);
                atomicAdd((unsigned long long *)&next->ent, (unsigned long long)L.ent);
                next->inc = 1u;
            }
        } else if (L.nq) {
            bfs_flush(L, next, nitems, (int32_t)L.nq, [&](int32_t i, int32_t &v, int32_t &p, int32_t &len) {
                v = L.pull.q[i];
                p = a.ce_ptr[v];
                len = a.ce_ptr[v + 1] - p;
            });
        }
    }
    for (int64_t w = (int64_t)gt + (int64_t)gridDim.x * BL_TPB; w < a.nwords; w += (int64_t)gridDim.x * BL_TPB) {
        const uint32_t f = F[w];
        if (f) a.vis[w] |= f;
        clr[w] = 0u;
    }
    if (nvb && t == 0 && L.nvb) atomicAdd(&next->nvb, L.nvb);
}

// Pull while the frontier holds few of the entries, as a forced path or an
// explicit th3 may ask: unreached rows would be read to their end, and the
// rows of a power-law graph that hold most entries lie next to each other
// (R-MAT 22, nine vertices in the frontier: 20 ms row by row).  Instead every
// wave streams an equal share of all entries; a column is tested in an LDS
// bitmap of the frontier (one bit per 1 << fold columns), and the hits, 64 at
// a time, are tested exactly and give each unreached row its smallest column.
// k_bfs_level follows and does the rest of the level.
constexpr int BS_BITMAP_WORDS = 8192;
constexpr int BS_QUEUE = 128;

__device__ __forceinline__ void seg_min_step(uint32_t &v, uint32_t key, uint32_t pv, uint32_t pk)
{
    if (pk == key) v = min(v, pv);
}

__global__ __launch_bounds__(BL_TPB, 8) void k_bfs_stream(BfsArgs a, int32_t l, int32_t fold)
{
    __shared__ uint32_t bm[BS_BITMAP_WORDS];
    __shared__ uint32_t q_col[BL_WAVES][BS_QUEUE], q_ord[BL_WAVES][BS_QUEUE];
    __shared__ uint64_t s_ent;
    __shared__ uint32_t s_found, s_nvb;
    const int t = threadIdx.x, lane = lane_id(), wv = wave_id();
    const BfsCount c = a.cnt[l % 3];
    if ((uint32_t)(c.items >> EV_TASK_BITS) + c.extra == 0 || !bfs_stream(a, c)) return;
    if (a.policy == 0 && (double)c.nvb < a.th3n) return;  // (push)
    BfsCount *next = &a.cnt[(l + 1) % 3];
    const uint32_t *F = a.bits[l % 3];
    uint32_t *nb = a.bits[(l + 1) % 3];
    for (int32_t i = t; i < BS_BITMAP_WORDS; i += BL_TPB) bm[i] = 0u;
    if (t == 0) {
        s_found = s_nvb = 0;
        s_ent = 0;
    }
    __syncthreads();
    for (int32_t w = t; w < a.nwords; w += BL_TPB) {
        uint32_t b = F[w];
        while (b) {
            const uint32_t i = ((uint32_t)w * 32u + (uint32_t)ctz32(b)) >> fold;
            b &= b - 1u;
            atomicOr(&bm[i >> 5], 1u << (i & 31));
        }
    }
    __syncthreads();
    const int64_t W = (int64_t)gridDim.x * BL_WAVES, wid = (int64_t)wv * gridDim.x + blockIdx.x;
    const int32_t c0 = (int32_t)(wid * a.nchunk / W), c1 = (int32_t)((wid + 1) * a.nchunk / W);
    uint32_t *qc = q_col[wv], *qo = q_ord[wv];
    uint32_t cnt = 0, head = 0, nfound = 0;
    int64_t ents = 0;
    auto flush = [&](uint32_t n) {
        const bool on = (uint32_t)lane < n;
        const uint32_t at = (head + (uint32_t)lane) & (BS_QUEUE - 1);
        const uint32_t o = on ? qo[at] : 0xFFFFFFFFu, col = on ? qc[at] : 0u;
        const int32_t v = on ? a.row[o] : 0;
        const bool seen = bit_of(a.vis, (uint32_t)v) || bit_of(F, (uint32_t)v);
        uint32_t m = on && !seen && bit_of(F, col) ? col : 0xFFFFFFFFu;
        seg_min_step(m, o, dpp_mov<dppc::ROW_SHR + 1>(~0u, m), dpp_mov<dppc::ROW_SHR + 1>(~o, o));
        seg_min_step(m, o, dpp_mov<dppc::ROW_SHR + 2>(~0u, m), dpp_mov<dppc::ROW_SHR + 2>(~o, o));
        seg_min_step(m, o, dpp_mov<dppc::ROW_SHR + 4>(~0u, m), dpp_mov<dppc::ROW_SHR + 4>(~o, o));
        seg_min_step(m, o, dpp_mov<dppc::ROW_SHR + 8>(~0u, m), dpp_mov<dppc::ROW_SHR + 8>(~o, o));
        seg_min_step(m, o, dpp_mov<dppc::ROW_BCAST15, 0xA>(~0u, m), dpp_mov<dppc::ROW_BCAST15, 0xA>(~o, o));
        seg_min_step(m, o, dpp_mov<dppc::ROW_BCAST31, 0xC>(~0u, m), dpp_mov<dppc::ROW_BCAST31, 0xC>(~o, o));
        const uint32_t on1 = dpp_mov<dppc::WF_SL1>(o, o);  // (with every lane active)
        const bool last = on && ((uint32_t)lane + 1 == n || on1 != o);
        if (last && m != 0xFFFFFFFFu && atomicMin(&a.parent[v], m) == 0xFFFFFFFFu) {
            a.level[v] = l + 1;
            const uint32_t old = atomicOr(&nb[v >> 5], 1u << (v & 31));
            if (!((old >> (v & 16)) & 0xFFFFu)) atomicAdd(&s_nvb, 1u);
            ents += a.rowinfo[v + 1].x - a.rowinfo[v].x;
            ++nfound;
        }
        head = (head + n) & (BS_QUEUE - 1);
        cnt -= n;
    };
    const uint64_t upto = lane == WAVE - 1 ? ~0ull : (1ull << (lane + 1)) - 1ull;
    int32_t ord = c0 < c1 ? a.chord[c0] : 0;
    for (int32_t ch = c0; ch < c1; ++ch) {
        uint32_t w[RE_CHUNK / WAVE];
#pragma unroll
        for (int j = 0; j < RE_CHUNK / WAVE; ++j) w[j] = a.col[(int64_t)ch * RE_CHUNK + j * WAVE + lane];
#pragma unroll
        for (int j = 0; j < RE_CHUNK / WAVE; ++j) {
            const int64_t e = (int64_t)ch * RE_CHUNK + j * WAVE + lane;
            const uint64_t starts = ballot((w[j] & RE_START) != 0u);
            const uint32_t o = (uint32_t)(ord + (int32_t)__popcll(starts & upto));
            ord += (int32_t)__popcll(starts);
            const uint32_t col = w[j] & ~RE_START, bit = col >> fold;
            const bool hit = ((bm[bit >> 5] >> (bit & 31)) & 1u) && e < a.nnz;
            const uint64_t h = ballot(hit);
            if (!h) continue;
            if (hit) {
                const uint32_t at = (head + cnt + (uint32_t)__popcll(h & (upto >> 1))) & (BS_QUEUE - 1);
                qo[at] = o;
                qc[at] = col;
            }
            cnt += (uint32_t)__popcll(h);
            if (cnt >= WAVE) {
                wave_lds_sync();
                flush(WAVE);
                wave_lds_sync();
            }
        }
    }
    wave_lds_sync();
    if (cnt) flush(cnt);
    ents = wave_sum(ents);
    nfound = wave_sum(nfound);
    if (lane == 0 && nfound) {
        atomicAdd(&s_found, nfound);
        atomicAdd((unsigned long long *)&s_ent, (unsigned long long)ents);
    }
    __syncthreads();
    if (t == 0 && s_found) {
        atomicAdd(&next->extra, s_found);
        atomicAdd((unsigned long long *)&next->ent, (unsigned long long)s_ent);
        atomicAdd(&next->nvb, s_nvb);
        next->inc = 1u;
    }
}

// With an explicit th3 the next level may have to push whatever a pull level
// found: the items of an incomplete list, written from the bitmap.
__global__ __launch_bounds__(BL_TPB) void k_bfs_list(BfsArgs a, int32_t l)
{
    __shared__ BfsLds L;
    const BfsCount c = a.cnt[l % 3];
    if (!c.inc || !((double)c.nvb < a.th3n)) return;
    // every workgroup lists its share of the words; the counts go to a record
    // of their own, and k_bfs_list_done moves them
    BfsCount *to = &a.cnt[3];
    const uint32_t *F = a.bits[l % 3];
    const int t = threadIdx.x;
    if (t == 0) L.nq = 0;
    __syncthreads();
    for (int64_t w0 = (int64_t)blockIdx.x * 64; w0 < a.nwords; w0 += (int64_t)gridDim.x * 64) {
        const int64_t w = w0 + t / 16;
        uint32_t bits = w < a.nwords ? (F[w] >> ((t & 15) * 2)) & 3u : 0u;
        while (bits) {
            const int32_t v = (int32_t)(w * 32 + (t & 15) * 2 + ctz32(bits));
            bits &= bits - 1u;
            L.q.v[atomicAdd(&L.nq, 1u)] = v;
        }
        __syncthreads();
        bfs_flush(L, to, a.items[l & 1], (int32_t)L.nq, [&](int32_t i, int32_t &v, int32_t &p, int32_t &len) {
            v = L.q.v[i];
            p = a.ce_ptr[v];
            len = a.ce_ptr[v + 1] - p;
        });
        if (t == 0) L.nq = 0;
        __syncthreads();
    }
}
__global__ void k_bfs_list_done(BfsArgs a, int32_t l)
{
    BfsCount c = a.cnt[l % 3];
    if (!c.inc || !((double)c.nvb < a.th3n)) return;
    c.items = a.cnt[3].items;
    c.extra = a.cnt[3].extra;
    c.inc = 0u;
    c.ent = 0u;
    a.cnt[l % 3] = c;
    a.cnt[3] = BfsCount{};
}

// Level 0: levels and parents unset but the source's, the frontier bitmap,
// item and counts of the source, rows without entries counted as reached (no
// edge leads to them), the other bitmaps and counts cleared.
__global__ __launch_bounds__(256) void k_bfs_start(BfsArgs a, int32_t source, const uint32_t *__restrict__ row_occ)
{
    const int64_t stride = (int64_t)gridDim.x * 256, g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // (level and parent need not be 16-byte aligned)
    for (int64_t v = g; v < a.n; v += stride) {
        a.level[v] = v == source ? 0 : -1;
        a.parent[v] = v == source ? (uint32_t)source : 0xFFFFFFFFu;
    }
    for (int64_t w = g; w < a.nwords; w += stride) {
        const uint32_t sb = w == (source >> 5) ? 1u << (source & 31) : 0u;
        a.vis[w] = row_occ ? ~row_occ[w] : 0u;
        a.bits[0][w] = sb;
        a.bits[1][w] = 0u;
        a.bits[2][w] = 0u;
    }
    if (g == 0) {
        const int32_t p0 = a.ce_ptr[source], p1 = a.ce_ptr[source + 1];
        BfsCount c{};
        if (p1 > p0) {
            c.items = (1ull << EV_TASK_BITS) + (uint64_t)(p1 - p0);
            a.items[0][0] = make_int4(0, p0, source, 0);
        } else {
            c.extra = 1u;
        }
        c.nvb = 1u;
        a.cnt[0] = c;
        a.cnt[1] = BfsCount{};
        a.cnt[2] = BfsCount{};
        a.cnt[3] = BfsCount{};
        a.rec->levels = 0;
        a.rec->reached = 0;
    }
}

static BfsArgs bfs_args(const DevMatrix &A, const DevBfs &B, int32_t *level, int32_t *parent, int policy, double th3,
                        double push_share)
{
    BfsArgs a;
    a.rowinfo = A.re_info;
    a.col = A.re_col;
    a.row = A.re_row;
    a.chord = A.re_chord;
    a.nchunk = A.re_nchunk;
    a.stream = policy == PATH_PULL || (policy == 0 && th3 > 0.0) ? 1 : 0;
    a.ce_ptr = A.ce_ptr;
    a.ce_row = A.ce_row;
    a.n = A.n;
    a.nwords = (A.n + 31) / 32;
    a.vis = B.vis;
    for (int i = 0; i < 3; ++i) a.bits[i] = B.bits[i];
    for (int i = 0; i < 2; ++i) a.items[i] = B.items[i];
    a.cnt = B.cnt;
    a.rec = B.rec;
    a.level = level;
    a.parent = (uint32_t *)parent;
    a.policy = policy;
    a.th3n = th3 > 0.0 ? th3 * (double)A.nbc : 0.0;
    a.nnz = A.re_nnz;
    a.push_max = (int64_t)(push_share * (double)A.re_nnz);
    return a;
}

hipError_t launch_bfs_start(const DevMatrix &A, const DevBfs &B, int32_t source, int32_t *level, int32_t *parent,
                            hipStream_t s)
{
    const BfsArgs a = bfs_args(A, B, level, parent, 0, 0.0, 0.0);
    const dim3 g((uint32_t)std::min<int64_t>(((int64_t)A.n + 255) / 256, 4096)), b(256);
    hipLaunchKernelGGL(k_bfs_start, g, b, 0, s, a, source, A.row_occ);
    return hipGetLastError();
}

hipError_t launch_bfs_level(const DevMatrix &A, const DevBfs &B, int32_t l, int32_t *level, int32_t *parent,
                            int policy, double th3, double push_share, hipStream_t s)
{
    const BfsArgs a = bfs_args(A, B, level, parent, policy, th3, push_share);
    const int64_t want = std::max<int64_t>(((int64_t)A.n + BL_TPB - 1) / BL_TPB,
                                           ((int64_t)A.re_nnz + 8 * BL_TPB - 1) / (8 * BL_TPB));
    // Where every wave has rows to take (four per lane and turn) one workgroup
    // per compute unit: with two, more of them queue at the counters where
    // items are reserved (R-MAT 22 134-143 against 142-160 us by source, R-MAT
    // 21 107-117 / 111-132, 4M random rows of 6 348-382 / 348-417, stencils of
    // 1.1M and 2M rows within 2%).  Smaller graphs take two: a stencil of
    // 207,360 rows takes 980 us from one source and 1078 from another, with
    // one workgroup each 1010 and 1031.
    const bool four = A.n >= 4 * WAVE * (BL_WAVES * 256);
    const dim3 g((uint32_t)std::min<int64_t>(want, four ? 256 : 512)), b(BL_TPB);
    if (a.th3n > 0.0 && policy == 0 && l > 0) {
        hipLaunchKernelGGL(k_bfs_list, g, b, 0, s, a, l);
        hipLaunchKernelGGL(k_bfs_list_done, dim3(1), dim3(1), 0, s, a, l);
    }
    if (a.stream) {
        int32_t fold = 0;
        while (((int64_t)A.n >> fold) >= (int64_t)BS_BITMAP_WORDS * 32) ++fold;
        hipLaunchKernelGGL(k_bfs_stream, dim3((uint32_t)std::min<int32_t>(A.re_nchunk, 512)), b, 0, s, a, l, fold);
    }
    if (four) hipLaunchKernelGGL(k_bfs_level<4>, g, b, 0, s, a, l);
    else hipLaunchKernelGGL(k_bfs_level<1>, g, b, 0, s, a, l);
    return hipGetLastError();
}

}  // namespace dbs
