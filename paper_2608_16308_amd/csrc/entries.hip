// gfx950 kernels over the entry views: the traversals of matrices whose
// entries sit in short COO blocks (graphs, relabelled meshes, heavily pruned
// layers), where a block's slot, descriptor and record words outweigh its one
// or two entries.
//
//   k_entry_scatter  vector blocker (densified x, masks) that also lists the
//                    columns of x as push work items
//   k_entry_push     y = A x over the column-entry view of the listed columns
//   k_entry_pull     y = A x by streaming the row-entry view; with the choice
//                    open, every workgroup takes it from the blocker's counts
//                    and pushes instead where it says so
//   k_ce_*           the column-entry view from the row-entry view, at upload
#include <algorithm>
#include <climits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace dbs {

template <int MODE> __host__ __device__ constexpr bool ev_valued() { return MODE == M_F32 || MODE == M_F16; }

// Raw x and value words, and the number they hold.
template <int MODE> __device__ __forceinline__ uint32_t ev_raw(const void *p, uint32_t i)
{
    if constexpr (MODE == M_F32) return ((const uint32_t *)p)[i];
    else return ((const uint16_t *)p)[i];
}
template <int MODE> __device__ __forceinline__ double ev_num(uint32_t raw)
{
    if constexpr (MODE == M_F32) return (double)__uint_as_float(raw);
    else return (double)h2f((uint16_t)raw);
}
// Product of a stored value and an x entry: exact in fp64, and never -0 (a
// row of such products sums to +0).
template <int MODE> __device__ __forceinline__ double ev_mul(uint32_t v, uint32_t x)
{
    return ev_num<MODE>(v) * ev_num<MODE>(x) + 0.0;
}
__device__ __forceinline__ bool ev_admit(const uint32_t *omask, int32_t complement, int32_t row)
{
    return !omask || ((omask[row >> 5] >> (row & 31)) & 1u) != (complement ? 1u : 0u);
}

// ---------------------------------------------------------------------------
// vector blocker with push work items
// ---------------------------------------------------------------------------
// The values and mask bits of k_scatter; besides, every distinct index whose
// column holds entries becomes a work item {first task, entry - first task,
// x bits, 0}, its tasks being the column's entries.  A workgroup reserves its
// items and tasks with one 64-bit atomic, so that
// items ascend in their first tasks without a scan over the workgroups.  A
// repeated index keeps the occurrence whose mask atomic found its bit clear.
// COUNT: the nonzero vector blocks and the distinct indices are added up in
// C_ECOUNT, from what the mask atomics found, so that the traversal can choose
// without reading the masks.
constexpr int ES_TPB = 256;

template <int MODE, bool COUNT>
__global__ __launch_bounds__(ES_TPB) void k_entry_scatter(const int32_t *__restrict__ xi, const void *__restrict__ xv,
                                                          int32_t k, int32_t n, void *__restrict__ xd,
                                                          uint32_t *__restrict__ xmask,
                                                          const int32_t *__restrict__ ce_ptr, int4 *__restrict__ items,
                                                          int32_t *__restrict__ counters)
{
    __shared__ uint64_t s_tot[ES_TPB / WAVE], s_cnt[ES_TPB / WAVE];
    __shared__ uint64_t s_base;
    const int32_t t = blockIdx.x * ES_TPB + threadIdx.x;
    const int lane = lane_id(), wv = wave_id();
    int32_t j = -1;
    uint32_t x = 0;
    if (t < k) {
        j = xi[t];
        if constexpr (ev_valued<MODE>()) x = ev_raw<MODE>(xv, (uint32_t)t);
    }
    const bool ok = t < k && j >= 0 && j < n;
    const uint64_t bad = ballot(t < k && !ok);
    if (lane == 0 && bad) atomicAdd(&counters[C_XBAD], (int32_t)__popcll(bad));
    int32_t p0 = 0, p1 = 0;
    if (ok) {
        p0 = ce_ptr[j];
        p1 = ce_ptr[j + 1];
        // an input equal to the absent-entry marker becomes the canonical NaN
        if constexpr (MODE == M_F32) {
            x = x == 0xFFFFFFFFu ? 0x7FC00000u : x;
            ((uint32_t *)xd)[j] = x;
        }
        if constexpr (MODE == M_F16) {
            x = x == 0xFFFFu ? 0x7E00u : x;
            ((uint16_t *)xd)[j] = (uint16_t)x;
        }
    }
    // runs of consecutive lanes with one mask word: one returning atomic each
    const uint32_t w = ok ? (uint32_t)j >> 5 : 0xFFFFFFFFu;
    const uint32_t bit = ok ? 1u << (j & 31) : 0u;
    const uint32_t wp = dpp_mov<dppc::WF_SR1>(~w, w);  // (every lane active, here and below)
    const bool head = lane == 0 || wp != w;
    const uint64_t heads = ballot(head);
    const uint64_t upto = lane == WAVE - 1 ? ~0ull : (1ull << (lane + 1)) - 1ull;
    const uint32_t run = (uint32_t)__popcll(heads & upto);
    const uint32_t incl = wave_run_or(bit, run);
    const uint32_t ip = dpp_mov<dppc::WF_SR1>(0u, incl);
    const uint32_t excl = head ? 0u : ip;
    const uint64_t above = heads & ~upto;
    const int last = above ? ctz64(above) - 1 : WAVE - 1;
    uint32_t old = 0;
    if (ok && lane == last) old = atomicOr(&xmask[w], incl);
    if constexpr (COUNT) {
        // the vector blocks that this run's atomic made nonzero
        const uint32_t was = ok && lane == last ? old : 0xFFFFFFFFu;
        const uint64_t lo = ballot(!(was & 0xFFFFu) && (incl & 0xFFFFu));
        const uint64_t hi = ballot(!(was >> 16) && (incl >> 16));
        if (lane == 0) s_cnt[wv] = (uint64_t)(__popcll(lo) + __popcll(hi));
    }
    old = (uint32_t)__shfl((int)old, last, WAVE);
    const bool first = ok && !((old | excl) & bit), own = first && p1 > p0;
    if constexpr (COUNT) {
        const uint64_t distinct = ballot(first);
        if (lane == 0) s_cnt[wv] |= (uint64_t)__popcll(distinct) << 32;
    }
    const uint64_t mine = own ? (1ull << EV_TASK_BITS) + (uint64_t)(p1 - p0) : 0ull;
    uint64_t inc = mine;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const uint64_t v = (uint64_t)__shfl_up((unsigned long long)inc, o, WAVE);
        if (lane >= o) inc += v;
    }
    if (lane == WAVE - 1) s_tot[wv] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t tot = 0;
#pragma unroll
        for (int i = 0; i < ES_TPB / WAVE; ++i) tot += s_tot[i];
        s_base = tot ? (uint64_t)atomicAdd((unsigned long long *)&counters[C_EITEMS], (unsigned long long)tot) : 0ull;
    }
    if constexpr (COUNT) {
        if (threadIdx.x == WAVE) {
            uint64_t cnt = 0;
#pragma unroll
            for (int i = 0; i < ES_TPB / WAVE; ++i) cnt += s_cnt[i];
            if (cnt) atomicAdd((unsigned long long *)&counters[C_ECOUNT], (unsigned long long)cnt);
        }
    }
    __syncthreads();
    if (own) {
        uint64_t at = s_base + inc - mine;
        for (int i = 0; i < wv; ++i) at += s_tot[i];
        const int32_t first = (int32_t)(at & ((1ull << EV_TASK_BITS) - 1));
        items[at >> EV_TASK_BITS] = make_int4(first, p0 - first, (int32_t)x, 0);
    }
}

// ---------------------------------------------------------------------------
// push over the column-entry view
// ---------------------------------------------------------------------------
struct EntryPushArgs {
    const int32_t *row;   // column-entry view: rows and values
    const void *val;
    const int4 *items;
    const uint32_t *omask;
    int32_t complement;
    double *yacc;
    uint32_t *ybits;
    int32_t *counters;
};

// 64 tasks (entries) per wave step, a task per lane, waves grid-stride.  The
// step's first item is found by a 64-ary search over the items' first tasks;
// the 64 items from there are held a lane each, and every lane finds its own
// by a six-step search through shuffles (an item has at least one task).
//
// Bound: by the chain of loads, and by atomics that meet in one word, which
// the memory serves one after the other: a power-law matrix's long rows are
// neighbours, so a mask atomic per entry put hundreds into each of the first
// words.  With one per first product of a row the pass takes 8.8 instead of 13.0 us
// (2^20 rows, 16 entries each, 1048 columns).
template <int MODE>
__device__ __forceinline__ void entry_push(const EntryPushArgs &a, int64_t gw, int64_t nw)
{
    const int lane = lane_id();
    const uint64_t all = *(const uint64_t *)&a.counters[C_EITEMS];
    const int32_t NT = (int32_t)(all >> EV_TASK_BITS), T = (int32_t)(all & ((1ull << EV_TASK_BITS) - 1));
    for (int64_t u = gw; u * WAVE < T; u += nw) {
        const int32_t t0 = (int32_t)(u * WAVE), t = t0 + lane;
        int32_t lo = 0, hi = NT;
        while (hi - lo > 1) {
            const int32_t step = (hi - lo + WAVE - 1) / WAVE, pi = lo + lane * step;
            const int32_t v = pi < hi ? a.items[pi].x : INT_MAX;
            const int L = 63 - __builtin_clzll(ballot(v <= t0));  // lane 0 probes lo: always set
            lo += L * step;
            hi = min(hi, lo + step);
        }
        const int4 it = lo + lane < NT ? a.items[lo + lane] : make_int4(INT_MAX, 0, 0, 0);
        int s = 0;
#pragma unroll
        for (int st = 32; st > 0; st >>= 1) {
            const int32_t v = __shfl(it.x, s + st, WAVE);
            if (s + st < WAVE && v <= t) s += st;
        }
        const int32_t e = __shfl(it.y, s, WAVE) + t;
        const uint32_t x = (uint32_t)__shfl(it.z, s, WAVE);
        if (t < T) {
            const int32_t row = a.row[e];
            uint32_t v = 0;
            if constexpr (ev_valued<MODE>()) v = ev_raw<MODE>(a.val, (uint32_t)e);
            if (ev_admit(a.omask, a.complement, row)) {
                // The first product of a row finds the sum 0 and marks the
                // row; so does one that finds it 0 again, which is harmless.
                bool mark = true;
                if constexpr (ev_valued<MODE>()) mark = atomicAdd(&a.yacc[row], ev_mul<MODE>(v, x)) == 0.0;
                if (mark) atomicOr(&a.ybits[row >> 5], 1u << (row & 31));
            }
        }
    }
}

constexpr int EPUSH_TPB = 256;
template <int MODE>
__global__ __launch_bounds__(EPUSH_TPB) void k_entry_push(EntryPushArgs a)
{
    entry_push<MODE>(a, (int64_t)blockIdx.x * (EPUSH_TPB / WAVE) + wave_id(),
                     (int64_t)gridDim.x * (EPUSH_TPB / WAVE));
}

// ---------------------------------------------------------------------------
// pull over the row-entry view
// ---------------------------------------------------------------------------
// Every wave streams an equal share of the entries (whole chunks), 64
// consecutive ones per step, a column word per lane.  A word's column is
// tested in an LDS bitmap of the stored x indices (one bit per 1 << fold
// columns: 128 KB of bitmap cover 2^20 columns without folding); the words
// that hit are queued in LDS with their entry position and row (rows are
// counted from the start marks: a ballot and a popcount), and every 64 queued
// hits are multiplied at once: value, x and row loads go out together, the
// products are summed in fp64 over the runs of one row by a segmented scan
// over the lanes, and a row is written when its run ends.  The last open run
// is carried to the next 64 hits, so a row inside one wave's share is written
// once, by a plain store; only the rows shared with the neighbouring waves'
// shares need atomics.
//
// Bound: the stream of the column words (4 bytes per entry, once per call,
// whatever x), then the hits' values and x gathers.
constexpr int EP_TPB = 1024;
constexpr int EP_WAVES = EP_TPB / WAVE;
constexpr int EP_QUEUE = 128;              // queued hits per wave (a step adds up to 64 to at most 63)
constexpr int32_t EP_BITMAP_WORDS = 32768; // LDS bitmap at most
constexpr int EP_STEPS = RE_CHUNK / WAVE;

struct EntryPullArgs {
    const uint32_t *col;
    const void *val;
    const int32_t *row;
    const int32_t *chord;
    int32_t nnz, nchunk;
    const void *xd;
    const uint32_t *xmask;
    int32_t nxw;      // 32-column mask words of x
    int32_t fold;     // log2 columns per bitmap bit
    int32_t nbw;      // bitmap words
    const uint32_t *omask;
    int32_t complement;
    double *yacc;
    uint32_t *ybits;  // NULL: dense output
    int32_t *counters;
    int32_t scanned;  // a scan ran: its choice decides whether there is work
    // open choice (DECIDE): the selector's numbers and the push side
    int32_t nbc;
    double th3, th3s;
    EntryPushArgs push;
};

extern __shared__ uint32_t ep_bits[];

// Halves a word's resolution: bit i of the result is bit 2 i or bit 2 i + 1.
__device__ __forceinline__ uint32_t fold_once(uint32_t w)
{
    w = (w | (w >> 1)) & 0x55555555u;
    w = (w | (w >> 1)) & 0x33333333u;
    w = (w | (w >> 2)) & 0x0F0F0F0Fu;
    w = (w | (w >> 4)) & 0x00FF00FFu;
    return (w | (w >> 8)) & 0xFFFFu;
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ void seg_step(double &sum, uint32_t &ok, uint32_t key)
{
    const uint32_t pk = dpp_mov<CTRL, ROW_MASK>(~key, key);
    const uint64_t u = (uint64_t)__double_as_longlong(sum);
    const uint32_t lo = dpp_mov<CTRL, ROW_MASK>(0u, (uint32_t)u), hi = dpp_mov<CTRL, ROW_MASK>(0u, (uint32_t)(u >> 32));
    const uint32_t pok = dpp_mov<CTRL, ROW_MASK>(0u, ok);
    if (pk == key) {
        sum += __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
        ok |= pok;
    }
}

// Copies the masks into the LDS bitmap, 16 bytes per load and BM_U loads in
// flight per thread.
constexpr int BM_U = 8;
__device__ __forceinline__ void ep_bitmap(const EntryPullArgs &a)
{
    const int t = threadIdx.x;
    const int32_t nq = (a.nxw + 3) >> 2;  // groups of four mask words
    for (int32_t q0 = 0; q0 < nq; q0 += BM_U * EP_TPB) {
        uint4 v[BM_U];
#pragma unroll
        for (int u = 0; u < BM_U; ++u) {
            const int32_t q = q0 + u * EP_TPB + t;
            v[u] = make_uint4(0, 0, 0, 0);
            if (4 * q + 3 < a.nxw) {
                v[u] = ((const uint4 *)a.xmask)[q];
            } else if (4 * q < a.nxw) {
                v[u].x = a.xmask[4 * q];
                if (4 * q + 1 < a.nxw) v[u].y = a.xmask[4 * q + 1];
                if (4 * q + 2 < a.nxw) v[u].z = a.xmask[4 * q + 2];
            }
        }
#pragma unroll
        for (int u = 0; u < BM_U; ++u) {
            const int32_t q = q0 + u * EP_TPB + t;
            if (q >= nq) continue;
            const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
            if (a.fold == 0) {
                ((uint4 *)ep_bits)[q] = v[u];
            } else if (a.fold == 1) {
                ((uint2 *)ep_bits)[q] = make_uint2(fold_once(w[0]) | fold_once(w[1]) << 16,
                                                   fold_once(w[2]) | fold_once(w[3]) << 16);
            } else {
                // 128 >> fold bits of one word
                uint32_t b = fold_once(fold_once(w[0])) | fold_once(fold_once(w[1])) << 8 |
                             fold_once(fold_once(w[2])) << 16 | fold_once(fold_once(w[3])) << 24;
                for (int32_t f = 2; f < a.fold; ++f) b = fold_once(b);
                const int64_t at = ((int64_t)q * 128) >> a.fold;
                if (b) atomicOr(&ep_bits[at >> 5], b << (at & 31));
            }
        }
    }
}

// DECIDE: push or pull was not settled on the host.  Every workgroup applies
// the selector's rule (Sec. 3.3.1 and the spread rule, as k_scan) to the
// blocker's counts before it copies the masks, so that no scan and no second
// traversal kernel is launched.  (Counting while the masks are copied made
// every push wait for the copy: 30 of 64 us with 4M columns.)
template <int MODE, bool DECIDE>
__global__ __launch_bounds__(EP_TPB) void k_entry_pull(EntryPullArgs a)
{
    constexpr bool VAL = ev_valued<MODE>();
    __shared__ uint32_t q_col[EP_WAVES][EP_QUEUE], q_ent[EP_WAVES][VAL ? EP_QUEUE : 1];
    __shared__ uint32_t q_ord[EP_WAVES][EP_QUEUE];
    const int t = threadIdx.x, lane = lane_id(), wv = wave_id();
    // the wave's chunks; its first words go out before the bitmap is formed
    const int64_t W = (int64_t)gridDim.x * EP_WAVES, wid = (int64_t)wv * gridDim.x + blockIdx.x;
    const int32_t c0 = (int32_t)(wid * a.nchunk / W), c1 = (int32_t)((wid + 1) * a.nchunk / W);
    uint32_t w[EP_STEPS];
#pragma unroll
    for (int j = 0; j < EP_STEPS; ++j)
        w[j] = c0 < c1 ? __builtin_nontemporal_load(&a.col[(int64_t)c0 * RE_CHUNK + j * WAVE + lane]) : 0u;
    int32_t ord = c0 < c1 ? a.chord[c0] : 0;
    if (a.scanned && a.counters[C_PATH] != PATH_PULL) return;
    if constexpr (DECIDE) {
        const uint64_t cnt = *(const uint64_t *)&a.counters[C_ECOUNT];
        const uint32_t N = (uint32_t)cnt, P = (uint32_t)(cnt >> 32);
        const bool spread = a.th3s > 0.0 && (int64_t)P < 2 * (int64_t)N && (double)N < a.th3s * (double)a.nbc;
        if ((double)N < a.th3 * (double)a.nbc || spread) {
            entry_push<MODE>(a.push, wid, W);
            return;
        }
    }
    if (a.fold > 1) {
        for (int32_t i = t; i < a.nbw; i += EP_TPB) ep_bits[i] = 0u;
        __syncthreads();
    }
    ep_bitmap(a);
    __syncthreads();
    if (c0 >= c1) return;

    uint32_t *qc = q_col[wv], *qe = q_ent[wv], *qo = q_ord[wv];
    uint32_t cnt = 0, head = 0;
    const uint32_t first = (uint32_t)ord;  // a run of this row may have begun in the share before
    // the open run: its row's index (NONE: no run), row, sum and whether a
    // stored, admitted product reached it
    constexpr uint32_t NONE = 0xFFFFFFFEu;
    uint32_t run = NONE, run_ok = 0;
    int32_t run_row = 0;
    double run_sum = 0.0;
    auto put = [&](bool on, uint32_t o, int32_t row, double v, bool shared) {
        if constexpr (VAL) {
            if (on) {
                if (shared || o == first) atomicAdd(&a.yacc[row], v);
                else a.yacc[row] = v;
            }
        }
    };
    // y structure (none for a dense output: atomics on one line take turns at
    // about 8 ns, and 5003 rows of 350 entries share few lines -- 27 us with
    // them, 10 without; testing the word before the atomic tripled the time of
    // a Boolean step on R-MAT 18)
    auto mark = [&](int32_t w, uint32_t bits) { atomicOr(&a.ybits[w], bits); };
    // the first n queued hits
    auto flush = [&](uint32_t n) {
        const bool on = (uint32_t)lane < n;
        const uint32_t at = (head + (uint32_t)lane) & (EP_QUEUE - 1);
        uint32_t o = on ? qo[at] : 0xFFFFFFFFu;
        uint32_t vr = 0, xr = 0;
        const int32_t row = on ? a.row[o] : 0;
        const uint32_t c = on ? qc[at] : 0u;
        if constexpr (VAL) {
            const uint32_t e = on ? qe[at] : 0u;
            vr = on ? ev_raw<MODE>(a.val, e) : 0u;
            xr = on ? ev_raw<MODE>(a.xd, c) : 0u;
        }
        uint32_t ok = on ? 1u : 0u;
        // a folded bit may stand for a neighbouring column
        if (a.fold) {
            if constexpr (VAL) ok = xr != (MODE == M_F32 ? 0xFFFFFFFFu : 0xFFFFu) ? ok : 0u;
            else ok = on ? (a.xmask[c >> 5] >> (c & 31)) & 1u : 0u;
        }
        if (on && !ev_admit(a.omask, a.complement, row)) ok = 0u;
        double sum = 0.0;
        if constexpr (VAL) sum = ok ? ev_mul<MODE>(vr, xr) : 0.0;
        // the open run goes on, or ends here
        const uint32_t o0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
        if (run == o0) {
            if (lane == 0) {
                sum += run_sum;
                ok |= run_ok;
            }
        } else if (run_ok) {
            put(lane == 0, run, run_row, run_sum, false);
            if (a.ybits && lane == 0) mark(run_row >> 5, 1u << (run_row & 31));
        }
        seg_step<dppc::ROW_SHR + 1>(sum, ok, o);
        seg_step<dppc::ROW_SHR + 2>(sum, ok, o);
        seg_step<dppc::ROW_SHR + 4>(sum, ok, o);
        seg_step<dppc::ROW_SHR + 8>(sum, ok, o);
        seg_step<dppc::ROW_BCAST15, 0xA>(sum, ok, o);
        seg_step<dppc::ROW_BCAST31, 0xC>(sum, ok, o);
        // runs that end before the last hit
        const uint32_t on1 = dpp_mov<dppc::WF_SL1>(o, o);
        const bool end = (uint32_t)lane + 1 < n && on1 != o;
        put(end && ok, o, row, sum, false);
        const uint32_t key = on ? (uint32_t)(row >> 5) : 0xFFFFFFFFu;
        const uint32_t bits = wave_run_or(end && ok ? 1u << (row & 31) : 0u, key);
        const uint32_t nkey = dpp_mov<dppc::WF_SL1>(~key, key);
        if (a.ybits && on && bits && nkey != key) mark((int32_t)key, bits);
        const int last = (int)n - 1;
        run = readlane_u32(o, last);
        run_row = (int32_t)readlane_u32((uint32_t)row, last);
        run_ok = readlane_u32(ok, last);
        run_sum = __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(sum), last));
        head = (head + n) & (EP_QUEUE - 1);
        cnt -= n;
    };
    const uint64_t upto = lane == WAVE - 1 ? ~0ull : (1ull << (lane + 1)) - 1ull;
    for (int32_t c = c0; c < c1; ++c) {
        uint32_t nw[EP_STEPS];
#pragma unroll
        for (int j = 0; j < EP_STEPS; ++j)
            nw[j] = c + 1 < c1 ? __builtin_nontemporal_load(&a.col[(int64_t)(c + 1) * RE_CHUNK + j * WAVE + lane]) : 0u;
#pragma unroll
        for (int j = 0; j < EP_STEPS; ++j) {
            const uint32_t e = (uint32_t)c * RE_CHUNK + j * WAVE + lane;
            const uint64_t starts = ballot((w[j] & RE_START) != 0u);
            const uint32_t o = (uint32_t)(ord + (int32_t)__popcll(starts & upto));
            ord += (int32_t)__popcll(starts);
            const uint32_t col = w[j] & ~RE_START;
            const uint32_t bit = col >> a.fold;
            const bool hit = ((ep_bits[bit >> 5] >> (bit & 31)) & 1u) && e < (uint32_t)a.nnz;
            const uint64_t h = ballot(hit);
            if (h) {
                if (hit) {
                    const uint32_t at = (head + cnt + (uint32_t)__popcll(h & (upto >> 1))) & (EP_QUEUE - 1);
                    qo[at] = o;
                    qc[at] = col;
                    if constexpr (VAL) qe[at] = e;
                }
                cnt += (uint32_t)__popcll(h);
                if (cnt >= WAVE) {
                    wave_lds_sync();
                    flush(WAVE);
                    wave_lds_sync();
                }
            }
        }
#pragma unroll
        for (int j = 0; j < EP_STEPS; ++j) w[j] = nw[j];
    }
    wave_lds_sync();
    if (cnt) flush(cnt);
    if (run != NONE && run_ok) {
        // the next share may go on with this row
        put(lane == 0, run, run_row, run_sum, true);
        if (a.ybits && lane == 0) mark(run_row >> 5, 1u << (run_row & 31));
    }
}

template <int MODE, bool DECIDE>
static hipError_t entry_pull(const EntryPullArgs &a, hipStream_t s)
{
    const size_t dyn = (size_t)a.nbw * 4;
    const int r = resident_workgroups((const void *)k_entry_pull<MODE, DECIDE>, EP_TPB, dyn);
    const int grid = std::max(1, std::min(r > 0 ? r : 256, (int)a.nchunk));
    hipLaunchKernelGGL((k_entry_pull<MODE, DECIDE>), dim3(grid), dim3(EP_TPB), dyn, s, a);
    return hipGetLastError();
}

static EntryPushArgs push_args(const DevMatrix &A, const DevCtx &C, const uint32_t *omask, int complement)
{
    EntryPushArgs a;
    a.row = A.ce_row;
    a.val = A.ce_val;
    a.items = C.items;
    a.omask = omask;
    a.complement = complement;
    a.yacc = C.yacc;
    a.ybits = C.ybits;
    a.counters = C.counters;
    return a;
}

static EntryPullArgs pull_args(const DevMatrix &A, const DevCtx &C, const uint32_t *omask, int complement)
{
    EntryPullArgs a;
    a.col = A.re_col;
    a.val = A.re_val;
    a.row = A.re_row;
    a.chord = A.re_chord;
    a.nnz = A.re_nnz;
    a.nchunk = A.re_nchunk;
    a.xd = C.xd;
    a.xmask = C.xmask;
    a.nxw = (A.nbc + 1) / 2;
    a.fold = 0;
    while (((a.nxw + (1 << a.fold) - 1) >> a.fold) > EP_BITMAP_WORDS) ++a.fold;
    // (whole 16-byte groups of mask words)
    a.nbw = std::max(1, (int)((((int64_t)(a.nxw + 3) / 4 * 128 >> a.fold) + 31) / 32));
    a.omask = omask;
    a.complement = complement;
    a.yacc = C.yacc;
    a.ybits = C.ybits;
    a.counters = C.counters;
    a.scanned = 0;
    a.nbc = A.nbc;
    a.th3 = a.th3s = 0.0;
    a.push = push_args(A, C, omask, complement);
    return a;
}

// The stream costs 4 bytes per entry whatever x is, and a fold of the bitmap
// lets columns next to x's through; the traversal of the blocks costs 10-20 us
// more to launch, 4 bytes per block, and the records of active vector blocks
// only.  With one or two entries per block the stream is faster at every size
// (1% clustered, 10% uniform x, us blocks / stream: R-MAT 22, 128M entries, 206 /
// 187, 958 / 517; 16M rows of 4 554 / 263, 1466 / 1306); with more of them up to
// a number of entries, beyond which a sparse x over many-entry blocks is better
// left to the blocks.  fp32, 6, 14 and 28 entries per block, the same x: 16M
// entries 52 / 52, 36 / 33, 37 / 30 and 121 / 104, 80 / 63, 74 / 49; 28-32M 105 /
// 94, 51 / 64, 42 / 48 and 201 / 234, 168 / 145, 110 / 94; 64M 176 / 179, 99 /
// 117, 58 / 93 and 398 / 578, 300 / 378, 298 / 250.  Boolean blocks read no value
// and pull at a cost per block: 4M entries 31 / 17, 32 / 17, 29 / 16; 7M (28 per
// block) 41 / 26; 16M 44 / 47, 36 / 29, 35 / 27 and, nearly every x, 68 / 115,
// 96 / 89, 92 / 79; 14M of a stencil in natural order with 1% of x in long runs
// 42 / 54.
bool entry_pull_pays(const DevMatrix &A, int mode)
{
    return A.re_nnz <= 2 * A.nblk || A.re_nnz <= ((mode == M_BOOL ? 8 : 15) << 20);
}

hipError_t launch_entry_pull(const DevMatrix &A, const DevCtx &C, int mode, const uint32_t *omask, int complement,
                             bool scanned, bool dense_out, hipStream_t s)
{
    EntryPullArgs a = pull_args(A, C, omask, complement);
    a.scanned = scanned ? 1 : 0;
    if (dense_out) a.ybits = nullptr;
    switch (mode) {
    case M_F32: return entry_pull<M_F32, false>(a, s);
    case M_F16: return entry_pull<M_F16, false>(a, s);
    case M_BOOL: return entry_pull<M_BOOL, false>(a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_entry_auto(const DevMatrix &A, const DevCtx &C, int mode, const uint32_t *omask, int complement,
                             double th3, double th3s, hipStream_t s)
{
    EntryPullArgs a = pull_args(A, C, omask, complement);
    a.th3 = th3;
    a.th3s = th3s;
    switch (mode) {
    case M_F32: return entry_pull<M_F32, true>(a, s);
    case M_F16: return entry_pull<M_F16, true>(a, s);
    case M_BOOL: return entry_pull<M_BOOL, true>(a, s);
    default: return hipErrorInvalidValue;
    }
}

template <bool COUNT>
static hipError_t entry_scatter(const DevMatrix &A, const DevCtx &C, int mode, int32_t k, const int32_t *x_idx,
                                const void *x_val, hipStream_t s)
{
    const dim3 g((k + ES_TPB - 1) / ES_TPB), b(ES_TPB);
    switch (mode) {
    case M_F32: hipLaunchKernelGGL((k_entry_scatter<M_F32, COUNT>), g, b, 0, s, x_idx, x_val, k, A.n, C.xd, C.xmask, A.ce_ptr, C.items, C.counters); break;
    case M_F16: hipLaunchKernelGGL((k_entry_scatter<M_F16, COUNT>), g, b, 0, s, x_idx, x_val, k, A.n, C.xd, C.xmask, A.ce_ptr, C.items, C.counters); break;
    default: hipLaunchKernelGGL((k_entry_scatter<M_BOOL, COUNT>), g, b, 0, s, x_idx, x_val, k, A.n, C.xd, C.xmask, A.ce_ptr, C.items, C.counters); break;
    }
    return hipGetLastError();
}

hipError_t launch_entry_scatter(const DevMatrix &A, const DevCtx &C, int mode, int32_t k, const int32_t *x_idx,
                                const void *x_val, bool count, hipStream_t s)
{
    if (k <= 0) return hipSuccess;
    return count ? entry_scatter<true>(A, C, mode, k, x_idx, x_val, s) : entry_scatter<false>(A, C, mode, k, x_idx, x_val, s);
}

hipError_t launch_entry_push(const DevMatrix &A, const DevCtx &C, int mode, const uint32_t *omask, int complement,
                             hipStream_t s)
{
    const EntryPushArgs a = push_args(A, C, omask, complement);
    const int64_t want = ((int64_t)A.re_nnz + EPUSH_TPB - 1) / EPUSH_TPB;
    const dim3 g((uint32_t)std::min<int64_t>(want, 2048)), b(EPUSH_TPB);
    switch (mode) {
    case M_F32: hipLaunchKernelGGL(k_entry_push<M_F32>, g, b, 0, s, a); break;
    case M_F16: hipLaunchKernelGGL(k_entry_push<M_F16>, g, b, 0, s, a); break;
    case M_BOOL: hipLaunchKernelGGL(k_entry_push<M_BOOL>, g, b, 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// column-entry view (at upload)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_ce_count(const uint32_t *__restrict__ col, int32_t nnz, int32_t *__restrict__ cnt)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * 256)
        atomicAdd(&cnt[col[e] & ~RE_START], 1);
}

// A wave per chunk; next[j]: the next free place of column j.
__global__ __launch_bounds__(256) void k_ce_fill(const uint32_t *__restrict__ col, const uint8_t *__restrict__ val,
                                                 int32_t vb, const int32_t *__restrict__ row,
                                                 const int32_t *__restrict__ chord, int32_t nnz, int32_t nchunk,
                                                 int32_t *__restrict__ next, int32_t *__restrict__ ce_row,
                                                 uint8_t *__restrict__ ce_val)
{
    const int lane = lane_id();
    const uint64_t upto = lane == WAVE - 1 ? ~0ull : (1ull << (lane + 1)) - 1ull;
    for (int32_t c = blockIdx.x * 4 + wave_id(); c < nchunk; c += gridDim.x * 4) {
        int32_t ord = chord[c];
        for (int j = 0; j < RE_CHUNK / WAVE; ++j) {
            const int64_t e = (int64_t)c * RE_CHUNK + j * WAVE + lane;
            const uint32_t w = col[e];
            const uint64_t starts = ballot((w & RE_START) != 0u);
            const int32_t o = ord + (int32_t)__popcll(starts & upto);
            ord += (int32_t)__popcll(starts);
            if (e >= nnz) continue;
            const int32_t p = atomicAdd(&next[w & ~RE_START], 1);
            ce_row[p] = row[o];
            if (vb == 4) ((uint32_t *)ce_val)[p] = ((const uint32_t *)val)[e];
            else if (vb == 2) ((uint16_t *)ce_val)[p] = ((const uint16_t *)val)[e];
        }
    }
}

hipError_t launch_ce_count(const DevMatrix &A, int32_t *cnt, hipStream_t s)
{
    hipLaunchKernelGGL(k_ce_count, dim3(2048), dim3(256), 0, s, A.re_col, A.re_nnz, cnt);
    return hipGetLastError();
}
hipError_t launch_ce_fill(const DevMatrix &A, int32_t vb, int32_t *next, int32_t *ce_row, void *ce_val, hipStream_t s)
{
    hipLaunchKernelGGL(k_ce_fill, dim3(2048), dim3(256), 0, s, A.re_col, (const uint8_t *)A.re_val, vb, A.re_row,
                       A.re_chord, A.re_nnz, A.re_nchunk, next, ce_row, (uint8_t *)ce_val);
    return hipGetLastError();
}

}  // namespace dbs
