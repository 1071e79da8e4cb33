// gfx950 pass for dense activations on the matrix cores: Y = A X for one to
// eight activations against a matrix whose blocks hold many entries (a pruned
// layer).
#include <algorithm>
#include <climits>

#include "device_common.hpp"
#include "kernels.hpp"

namespace dbs {

// Workgroups take block rows (or parts of one), their waves equal stretches of
// each class of its blocks (see DevMatrix: the list is ordered by class, so
// that a class's loop has no branch on the format); a block (16 rows x 16
// columns) times 16 columns x 16 tokens, of which up to 8 are used, is one
// v_mfma_f32_16x16x16_f16 or four v_mfma_f32_16x16x4_f32.  The fp32 block
// product is added to fp64 accumulators, four per lane, and the waves' sums
// are combined in LDS, so y is written by the pass and no other kernel runs.
//
// A operand: lane l holds row l % 16, columns 4 (l / 16) .. + 3 (fp32: its
// c-th column in the c-th product, the same columns of x beside them).  All
// loads are in memory order, whole lines (loading each lane's four values
// from where they start costs the address unit a cycle per lane: 45 us
// instead of 31 on 4096 x 14336 fp16, eight tokens), and cross-lane moves
// bring them to operand order.  In the row formats the row's stored entries
// among the four columns are consecutive in the value run: three words hold
// them, a shift aligns them and a byte permutation, with a selector per 4-bit
// pattern, moves them to their columns (fp32: through LDS and selects).
// ForceCSC blocks gather their entries; COO blocks are scattered into a tile
// in LDS, an entry per lane.
//
// Zeros stand for absent entries and inactive x, which only holds for finite
// numbers (0 * inf must not reach a sum): a wave whose sums are not all finite
// takes its blocks again, those whose own product is not finite with both
// masks.
//
// Bound: by the records streamed once, of which it reads a Dense block's
// values or a row format's masks, starts and run (4096 x 14336 fp16 half
// pruned, eight tokens: 97 MB in 27 us, 3.6 TB/s beside the 4.7 of a large
// copy); four kernels with a lane per row and a loop over the tokens took 94
// us, of 71 in the block pass.
struct BatchArgs {
    const int32_t *col;    // block list (see DevMatrix): block column, descriptor
    const uint64_t *desc;
    const int32_t *rptr;   // where each block row's classes begin
    const uint8_t *pay;
    const void *x;         // nb x n
    int32_t n, m, nb;
    void *y;               // nb x m
    float *y32;
    // a block row split over several workgroups: fp64 sums (zero between
    // calls) and the parts of each block row that have added theirs
    int32_t parts;
    double *yacc;
    int64_t ystride;
    int32_t *rdone;
};

typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

// Four consecutive values: words[0..1] (fp16) or words[0..3] (fp32), from a
// place aligned to the value only.
template <int VB> struct __attribute__((packed, aligned(VB))) Vals4 {
    uint32_t w[VB];
};
template <int VB> __device__ __forceinline__ uint32_t val_at(const uint8_t *vals, int32_t i)
{
    if constexpr (VB == 4) return ((const uint32_t *)vals)[i];
    else return ((const uint16_t *)vals)[i];
}
template <int VB> __device__ __forceinline__ float val_f(uint32_t raw)
{
    if constexpr (VB == 4) return __uint_as_float(raw);
    else return h2f((uint16_t)raw);
}
template <int VB> __device__ __forceinline__ void put4(uint32_t (&w)[VB], int i, uint32_t raw)
{
    if constexpr (VB == 4) w[i] = raw;
    else w[i >> 1] = (i & 1) ? w[i >> 1] | raw << 16 : raw;
}

constexpr int BD_U = 4;           // blocks in flight per wave
constexpr uint32_t RUN = MC_RUN;  // values of a row-format block, loaded as a run

// Byte selectors that move the first popc(nib) of four halves to the set
// positions of nib and zeros to the others (0x0C: constant 0).
__device__ __forceinline__ uint2 spread_sel(uint32_t nib)
{
    uint32_t s[2] = {0x0C0C0C0Cu, 0x0C0C0C0Cu};
    uint32_t k = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if ((nib >> c) & 1u) {
            const uint32_t two = (2u * k) | ((2u * k + 1u) << 8);
            s[c >> 1] = (s[c >> 1] & ~(0xFFFFu << (16 * (c & 1)))) | two << (16 * (c & 1));
            ++k;
        }
    }
    return make_uint2(s[0], s[1]);
}

// The same for four words: the first popc(nib) of v at the set positions.
__device__ __forceinline__ void spread4(uint32_t (&v)[4], uint32_t nib)
{
    const bool b0 = nib & 1u, b1 = nib & 2u, b2 = nib & 4u, b3 = nib & 8u;
    // entry c is v[number of set bits below c]
    const uint32_t a1 = b0 ? v[1] : v[0];
    const uint32_t a2 = b0 ? (b1 ? v[2] : v[1]) : (b1 ? v[1] : v[0]);
    const uint32_t k3 = __popc(nib & 7u);
    const uint32_t a3 = k3 & 2u ? (k3 & 1u ? v[3] : v[2]) : (k3 & 1u ? v[1] : v[0]);
    v[0] = b0 ? v[0] : 0u;
    v[1] = b1 ? a1 : 0u;
    v[2] = b2 ? a2 : 0u;
    v[3] = b3 ? a3 : 0u;
}

// The lane's four x of its token, at xb; RAG: zeros past the `left` columns
// the vector block has.
template <int VB, bool RAG>
__device__ __forceinline__ Vals4<VB> load_x4(const uint8_t *xb, int32_t left)
{
    if (RAG && left < BS) {
        const int32_t c0 = (lane_id() & 3) * 4;
        uint32_t w[VB];
#pragma unroll
        for (int i = 0; i < 4; ++i) put4<VB>(w, i, c0 + i < left ? val_at<VB>(xb, i) : 0u);
        Vals4<VB> v;
#pragma unroll
        for (int i = 0; i < VB; ++i) v.w[i] = w[i];
        return v;
    }
    return *(const Vals4<VB> *)xb;
}

// Lane r + 16 q takes what lane 4 r + q holds (memory order to operand order).
__device__ __forceinline__ uint32_t to_operand(uint32_t v, uint32_t src4)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)src4, (int)v);
}

// Entry (r, c) of a block: its raw value, or false.
template <int VB>
__device__ __forceinline__ bool entry_of(const uint8_t *rec, uint64_t d, uint32_t r, uint32_t c, uint32_t &raw)
{
    const uint32_t type = desc_type(d), nnz = desc_nnz(d);
    if (type == T_COO) {
        const uint32_t want = r << 4 | c;
        int32_t at = -1;  // (no way out of the loop but its end: lanes seek different entries)
        if (desc_inline(d)) {
            for (uint32_t e = 0; e < nnz; ++e)
                if (((uint32_t)(d >> inline_shift(e, VB)) & 0xFFu) == want) at = (int32_t)e;
            if (at < 0) return false;
            raw = (uint32_t)(d >> (inline_shift((uint32_t)at, VB) + 8u)) & (VB == 4 ? ~0u : 0xFFFFu);
        } else {
            for (uint32_t e = 0; e < nnz; ++e)
                if (rec[VB * nnz + e] == want) at = (int32_t)e;
            if (at < 0) return false;
            raw = val_at<VB>(rec, at);
        }
        return true;
    }
    const uint16_t *mk = (const uint16_t *)(rec + HDR_MASK);
    const uint32_t g = type == T_FCSC ? c : r, o = type == T_FCSC ? r : c, m = mk[g];
    if (!((m >> o) & 1u)) return false;
    const uint32_t at = type == T_DENSE ? r * BS + c : rec[HDR_START + g] + __popc(m & ((1u << o) - 1u));
    raw = val_at<VB>(rec + values_at(type, nnz), (int32_t)at);
    return true;
}

// One wave's walk over a stretch of one class of a block row's blocks.
template <int VB, bool RAG>
struct MfmaWalk {
    const BatchArgs &a;
    const uint8_t *xl;      // the lane's x in vector block 0
    uint8_t *tile;          // this wave's LDS: 256 values
    const uint2 *sel;
    double acc[4];
    uint32_t r, q, lane, src4;

    __device__ __forceinline__ Vals4<VB> x_of(int32_t J) const
    {
        return load_x4<VB, RAG>(xl + (int64_t)J * BS * VB, a.n - J * BS);
    }
    __device__ __forceinline__ static bool any_x(const Vals4<VB> &x)
    {
        uint32_t any = 0;
#pragma unroll
        for (int k = 0; k < VB; ++k) any |= x.w[k];
        return ballot((any & (VB == 4 ? 0x7FFFFFFFu : 0x7FFF7FFFu)) != 0u) != 0;
    }
    // False (CHECK only), and nothing added: the block's product is not finite.
    template <bool CHECK>
    __device__ __forceinline__ bool multiply(const uint32_t (&aw)[VB], const Vals4<VB> &x)
    {
        uint32_t xw[VB];
#pragma unroll
        for (int k = 0; k < VB; ++k) xw[k] = to_operand(x.w[k], src4);
        f4_t p = {0.f, 0.f, 0.f, 0.f};
        if constexpr (VB == 2) {
            p = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4_t, make_uint2(aw[0], aw[1])),
                                                      __builtin_bit_cast(h4_t, make_uint2(xw[0], xw[1])), p, 0, 0, 0);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                p = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(aw[k]), __uint_as_float(xw[k]), p, 0, 0, 0);
        }
        if constexpr (CHECK) {
            bool fin = true;
#pragma unroll
            for (int i = 0; i < 4; ++i) fin = fin && __builtin_isfinite(p[i]);
            if (ballot((int32_t)r < a.nb && !fin)) return false;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += (double)p[i];
        return true;
    }

    // One block with both masks: only products of a stored entry and an
    // active x are formed.  A lane holds the entries of row r in columns 4 q
    // .. + 3 and sums their products for one token after the other; the four
    // sums of a row go to the lane whose accumulators hold it.
    __device__ __forceinline__ void masked_block(int32_t J, uint64_t d)
    {
        const uint8_t *rec = a.pay + desc_off(d);
        uint32_t av[4], have = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            av[c] = 0u;
            if (entry_of<VB>(rec, d, r, q * 4 + (uint32_t)c, av[c])) have |= 1u << c;
        }
        for (int32_t tk = 0; tk < a.nb; ++tk) {
            const uint8_t *xp = (const uint8_t *)a.x + (int64_t)tk * a.n * VB;
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int32_t j = J * BS + (int32_t)q * 4 + c;
                const uint32_t xr = j < a.n ? val_at<VB>(xp, j) : 0u;
                if (((have >> c) & 1u) && (xr & (VB == 4 ? 0x7FFFFFFFu : 0x7FFFu)))
                    s = fmaf(val_f<VB>(av[c]), val_f<VB>(xr), s);
            }
            s += __shfl_xor(s, 16, WAVE);
            s += __shfl_xor(s, 32, WAVE);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = __shfl(s, (int)q * 4 + i, WAVE);
                if ((int32_t)r == tk) acc[i] += (double)v;
            }
        }
    }

    // Blocks b0 .. b1 - 1 of the list, CLASS their class; everything a group
    // of BD_U blocks needs is loaded while the group before it is multiplied:
    // x and the value array, both in memory order (whole lines), a row
    // format's row mask and start, a COO block's coordinates.  CHECK: blocks
    // whose product is not finite are taken with both masks.
    template <int CLASS, bool CHECK>
    __device__ __forceinline__ void walk(int32_t b0, int32_t b1)
    {
        constexpr int U = CHECK ? 2 : BD_U;  // (more would cost the first walk its registers)
        for (int32_t base = b0; base < b1; base += WAVE) {
            const int32_t nbk = min(WAVE, b1 - base);
            const int32_t Jl = (int32_t)lane < nbk ? a.col[base + lane] : 0;
            const uint64_t dl = (int32_t)lane < nbk ? a.desc[base + lane] : 0ull;
            const uint32_t nl = desc_nnz(dl);
            // byte offsets: record; values behind it
            const uint64_t ol = desc_off(dl);
            const uint32_t vl = CLASS == MC_ROWS ? values_at(desc_type(dl), nl) : 0u;
            uint32_t mn[U], en[U], vn[U][VB], nn[U];
            uint64_t dn[U];
            Vals4<VB> xn[U];
            auto fetch = [&](int32_t i0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = min(i0 + u, nbk - 1);
                    xn[u] = x_of((int32_t)readlane_u32((uint32_t)Jl, i));
                    const uint8_t *rec = a.pay + readlane_u64(ol, i);
                    if constexpr (CLASS == MC_DENSE) {
                        const Vals4<VB> v = ((const Vals4<VB> *)(rec + HDR_START))[lane];
#pragma unroll
                        for (int k = 0; k < VB; ++k) vn[u][k] = v.w[k];
                    } else if constexpr (CLASS == MC_ROWS) {
                        mn[u] = ((const uint16_t *)rec)[r];
                        en[u] = rec[HDR_START + r];
                        // VB / 2 words per lane: RUN values (what lies behind
                        // the block's own is not used; the payload is padded)
                        const uint32_t *vw = (const uint32_t *)(rec + readlane_u32(vl, i));
#pragma unroll
                        for (int k = 0; k < VB / 2; ++k) vn[u][k] = vw[lane * (VB / 2) + k];
                    } else if constexpr (CLASS == MC_COO) {
                        nn[u] = readlane_u32(nl, i);
                        dn[u] = readlane_u64(dl, i);
                        mn[u] = vn[u][0] = 0u;
                        if (desc_inline(dn[u])) {
                            if (lane < nn[u]) {
                                const uint32_t sh = inline_shift(lane, VB);
                                mn[u] = (uint32_t)(dn[u] >> sh) & 0xFFu;
                                vn[u][0] = (uint32_t)(dn[u] >> (sh + 8));
                            }
                        } else if (lane < nn[u]) {
                            mn[u] = rec[VB * nn[u] + lane];
                            vn[u][0] = val_at<VB>(rec, (int32_t)lane);
                        }
                    } else {
                        dn[u] = readlane_u64(dl, i);
                    }
                }
            };
            fetch(0);
            uint64_t masked = 0;
            for (int32_t i0 = 0; i0 < nbk; i0 += U) {
                uint32_t aw[U][VB];
                Vals4<VB> x[U];
                bool act[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    x[u] = xn[u];
                    act[u] = i0 + u < nbk && any_x(x[u]);
                    if (!act[u]) continue;
                    if constexpr (CLASS == MC_DENSE) {
#pragma unroll
                        for (int k = 0; k < VB; ++k) aw[u][k] = to_operand(vn[u][k], src4);
                    } else if constexpr (CLASS == MC_ROWS) {
                        // the lane's entries start at `at` in the value run
                        const uint32_t at = en[u] + __popc(mn[u] & ((1u << (q * 4)) - 1u)), nib = (mn[u] >> (q * 4)) & 15u;
                        if constexpr (VB == 2) {
                            const uint32_t s0 = (at >> 1) * 4, sh = (at & 1u) * 16u;
                            const uint32_t w0 = to_operand(vn[u][0], s0), w1 = to_operand(vn[u][0], s0 + 4),
                                           w2 = to_operand(vn[u][0], s0 + 8);
                            const uint32_t lo = __builtin_amdgcn_alignbit(w1, w0, sh),
                                           hi = __builtin_amdgcn_alignbit(w2, w1, sh);
                            const uint2 sl = sel[nib];
                            aw[u][0] = __builtin_amdgcn_perm(hi, lo, sl.x);
                            aw[u][1] = __builtin_amdgcn_perm(hi, lo, sl.y);
                        } else {
                            uint32_t *run = (uint32_t *)tile;
                            *(uint2 *)&run[lane * 2] = make_uint2(vn[u][0], vn[u][1]);
                            wave_lds_sync();
                            uint32_t w[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k) w[k] = run[(at + k) & (RUN - 1)];
                            wave_lds_sync();
                            spread4(w, nib);
#pragma unroll
                            for (int k = 0; k < 4; ++k) aw[u][k] = w[k];
                        }
                    } else if constexpr (CLASS == MC_COO) {
#pragma unroll
                        for (int k = 0; k < VB; ++k) ((uint32_t *)tile)[k * WAVE + lane] = 0u;
                        wave_lds_sync();
                        if (lane < nn[u]) {
                            if constexpr (VB == 4) ((uint32_t *)tile)[mn[u]] = vn[u][0];
                            else ((uint16_t *)tile)[mn[u]] = (uint16_t)vn[u][0];
                        }
                        wave_lds_sync();
#pragma unroll
                        for (int k = 0; k < VB; ++k) aw[u][k] = ((const uint32_t *)tile)[(r * 4 + q) * VB + k];
                        wave_lds_sync();
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            uint32_t raw = 0u;
                            if (!entry_of<VB>(a.pay + desc_off(dn[u]), dn[u], r, q * 4 + c, raw)) raw = 0u;
                            put4<VB>(aw[u], c, raw);
                        }
                    }
                }
                if (i0 + U < nbk) fetch(i0 + U);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (act[u] && !multiply<CHECK>(aw[u], x[u])) masked |= 1ull << (i0 + u);
            }
            if constexpr (CHECK) {
                for (; masked; masked &= masked - 1ull) {
                    const int i = ctz64(masked);
                    masked_block((int32_t)readlane_u32((uint32_t)Jl, i), readlane_u64(dl, i));
                }
            }
        }
    }

    template <bool CHECK> __device__ __forceinline__ void walk_all(const int32_t (&cb)[MC_COUNT][2])
    {
        walk<MC_DENSE, CHECK>(cb[MC_DENSE][0], cb[MC_DENSE][1]);
        walk<MC_ROWS, CHECK>(cb[MC_ROWS][0], cb[MC_ROWS][1]);
        walk<MC_COO, CHECK>(cb[MC_COO][0], cb[MC_COO][1]);
        walk<MC_OTHER, CHECK>(cb[MC_OTHER][0], cb[MC_OTHER][1]);
    }
};

template <int VB, int NW, bool RAG>
__global__ __launch_bounds__(NW *WAVE, VB == 2 ? 6 : 4) void k_rows_mfma(BatchArgs a)
{
    __shared__ double red[NW][16 * 8];
    __shared__ uint2 sel[16];
    __shared__ __align__(16) uint8_t tiles[NW][BS * BS * VB];
    const int t = threadIdx.x, lane = lane_id(), wv = wave_id();
    const uint32_t r = lane & 15, q = lane >> 4;
    const int32_t R = (int32_t)(blockIdx.x / (uint32_t)a.parts), part = (int32_t)(blockIdx.x % (uint32_t)a.parts);
    if (t < 16) sel[t] = spread_sel((uint32_t)t);
    __syncthreads();
    const bool tok = (int32_t)r < a.nb;
    // memory order: lane 4 i + p loads part p (four columns) of token i, or of
    // row i (a lane without a token loads the first one's x: its sums are not
    // used); operand order: lane r + 16 q holds part q of row or token r
    const uint32_t li = lane >> 2, lp = lane & 3;
    // (64 bits: eight tokens of 2^28 columns are 8 GB in fp32)
    const uint8_t *xl = (const uint8_t *)a.x + ((int32_t)li < a.nb ? (int64_t)li * a.n * VB : 0) + lp * 4 * VB;
    MfmaWalk<VB, RAG> w{a, xl, tiles[wv], sel, {0.0, 0.0, 0.0, 0.0}, r, q, (uint32_t)lane, (r * 4 + q) * 4};
    // the wave's share of each class of the block row's blocks
    int32_t cb[MC_COUNT][2];
#pragma unroll
    for (int k = 0; k < MC_COUNT; ++k) {
        const int32_t h0 = a.rptr[R * MC_COUNT + k], cnt = a.rptr[R * MC_COUNT + k + 1] - h0;
        const int32_t at = part * NW + wv, of = a.parts * NW;
        cb[k][0] = h0 + (int32_t)((int64_t)at * cnt / of);
        cb[k][1] = h0 + (int32_t)((int64_t)(at + 1) * cnt / of);
    }
    w.template walk_all<false>(cb);
    double (&acc)[4] = w.acc;
    // lane: rows 4 q + i, token r
    bool fin = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) fin = fin && __builtin_isfinite(acc[i]);
    if (ballot(tok && !fin)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = 0.0;
        w.template walk_all<true>(cb);
    }
    if (r < 8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wv][r * 16 + q * 4 + i] = acc[i];
    }
    __syncthreads();
    auto put = [&](int o, double s) {
        const int64_t row = (int64_t)R * BS + (o & 15);
        if (row >= a.m) return;
        const int64_t to = (int64_t)(o >> 4) * a.m + row;
        if constexpr (VB == 4) ((float *)a.y)[to] = (float)s;
        else ((uint16_t *)a.y)[to] = f64_to_f16_rne(s);
        if (a.y32) a.y32[to] = (float)s;
    };
    for (int o = t; o < 16 * a.nb; o += NW * WAVE) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < NW; ++k) s += red[k][o];
        if (a.parts == 1) put(o, s);
        else atomicAdd(&a.yacc[(int64_t)(o >> 4) * a.ystride + (int64_t)R * BS + (o & 15)], s);
    }
    if (a.parts == 1) return;
    // The adds are device-scope atomics, complete when the wave's memory
    // counter drains; the workgroup that counts the block row's last part
    // takes the sums, clearing them, by atomic exchanges.
    __shared__ int32_t s_last;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (t == 0) s_last = atomicAdd(&a.rdone[R], 1) == a.parts - 1 ? 1 : 0;
    __syncthreads();
    if (!s_last) return;
    for (int o = t; o < 16 * a.nb; o += NW * WAVE)
        put(o, atomicExch(&a.yacc[(int64_t)(o >> 4) * a.ystride + (int64_t)R * BS + (o & 15)], 0.0));
    if (t == 0) atomicExch(&a.rdone[R], 0);
}

bool rows_mfma_fits(const DevMatrix &A) { return A.ab_col != nullptr; }

// Launch shape.  A group of loads takes about 2 us whatever runs beside it, so
// what counts is the number of waves; the exchange of sums costs each part of
// a block row another 2 us or so.  Long block rows (128 blocks and more on
// average): up to 256 of them take 16 waves per workgroup, and several
// workgroups each while those fill the compute units once and every wave keeps
// four blocks; more take eight waves, and as many workgroups as the device
// holds at once.  fp16, eight tokens, us with 16 waves / with eight and as many
// as the device holds: 4096 x 14336 31 / 35, 700 x 7000 13 / 18, 3000 x 3000
// 15 / 22, 11008 x 4096 35 / 25, 5003 x 7001 37 / 26.
// Short block rows take four waves; where there are 2048 and more of at most 16
// blocks, one: a workgroup's launch and exchange then cost more than its
// blocks (four tokens, four waves / one: 10^6 x 16 fp16 137 / 48, fp32 207 /
// 65; 64000 x 256 fp32 24 / 19; at 2048 rows of 16 they are equal, with 1024
// rows or 32 blocks four are faster).
struct MfmaShape {
    int waves;
    int32_t parts;
};
static MfmaShape mfma_shape(const DevMatrix &A)
{
    if (A.nbr >= 2048 && A.nblk <= (int64_t)A.nbr * 16) return {1, 1};
    if (A.nbr <= 0 || A.nblk < (int64_t)A.nbr * 128) return {4, 1};
    const int waves = A.nbr <= 256 ? 16 : 8;
    // 8-wave workgroups per compute unit: 3 at no more than 80 registers
    // (fp16: see k_rows_mfma's launch bounds), 2 at no more than 128
    const int64_t hold = A.nbr <= 256 ? 256 : 256 * (A.dtype == 1 ? 3 : 2);
    const int64_t most = std::min<int64_t>(hold / A.nbr, A.nblk / ((int64_t)A.nbr * waves * 4));
    return {waves, (int32_t)std::max<int64_t>(1, std::min<int64_t>(most, 8))};
}
int32_t rows_mfma_parts(const DevMatrix &A) { return mfma_shape(A).parts; }

hipError_t launch_rows_mfma(const DevMatrix &A, const DevCtx &C, double *yacc, int32_t nb, const void *x, void *y,
                            float *y32, hipStream_t s)
{
    BatchArgs a;
    a.parts = rows_mfma_parts(A);
    a.yacc = yacc;
    a.ystride = (int64_t)A.nbr * BS;
    a.rdone = C.rdone;
    a.col = A.ab_col;
    a.desc = A.ab_desc;
    a.rptr = A.ab_rptr;
    a.pay = A.pay;
    a.x = x;
    a.n = A.n;
    a.m = A.m;
    a.nb = nb;
    a.y = y;
    a.y32 = y32;
    const int nw = mfma_shape(A).waves;
    const bool rag = A.n % BS != 0;
    const dim3 g((uint32_t)(A.nbr * a.parts)), b((uint32_t)(nw * WAVE));
#define DBS_MFMA(VB, NW, RAG) hipLaunchKernelGGL((k_rows_mfma<VB, NW, RAG>), g, b, 0, s, a)
#define DBS_MFMA_RAG(VB, NW)          \
    do {                              \
        if (rag) DBS_MFMA(VB, NW, true); \
        else DBS_MFMA(VB, NW, false); \
    } while (0)
    if (A.dtype == 1) {
        if (nw == 16) DBS_MFMA_RAG(2, 16);
        else if (nw == 8) DBS_MFMA_RAG(2, 8);
        else if (nw == 4) DBS_MFMA_RAG(2, 4);
        else DBS_MFMA_RAG(2, 1);
    } else {
        if (nw == 16) DBS_MFMA_RAG(4, 16);
        else if (nw == 8) DBS_MFMA_RAG(4, 8);
        else if (nw == 4) DBS_MFMA_RAG(4, 4);
        else DBS_MFMA_RAG(4, 1);
    }
#undef DBS_MFMA_RAG
#undef DBS_MFMA
    return hipGetLastError();
}

}  // namespace dbs
