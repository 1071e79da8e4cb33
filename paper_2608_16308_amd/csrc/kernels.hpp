// Host-side launch interface of the gfx950 kernels (implemented in kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dbs {

// Device-resident DB matrix (Sec. 3.2.1): dual block views over one payload.
//
// On the device the primary (block-CSR) order is laid out in pull-segment
// slots: segment s owns slots [16 s, 16 s + 16), its blocks in block-CSR
// order followed by padding (block column -1).  A pull lane thus finds its
// block column and descriptor at 16 s + lane without first reading the
// segment.  The block-CSC view holds each block's descriptor (csc_desc)
// next to its block row instead of its primary id, so that push reaches a
// block's record in one step.  The payload records are unchanged.
struct DevMatrix {
    int32_t m = 0, n = 0, nbr = 0, nbc = 0;
    int64_t nblk = 0, nseg = 0;
    int32_t dtype = 0;  // dbs_dtype
    const int32_t *sl_col = nullptr;    // 16 nseg: block column, -1 = padding, sign bit = non-COO (listed)
    const uint64_t *sl_desc = nullptr;  // 16 nseg: descriptor
    const uint32_t *seg_rs = nullptr;   // nseg: block row of the segment
    const int32_t *cb_ptr = nullptr;    // block-CSC view: column pointer (nbc + 1)
    const int32_t *csc_row = nullptr;   // block row per CSC position
    const uint64_t *csc_desc = nullptr; // descriptor per CSC position
    // The non-COO blocks in block-CSR order (pull takes them row-per-lane,
    // see pull_rows), cut into chunks of at most HV_CHUNK consecutive blocks
    // of one block row: chunk c holds list entries hv_cstart[c] ..
    // hv_cstart[c + 1] - 1 of block row hv_crow[c].
    const int32_t *hv_col = nullptr;     // nheavy: block column
    const uint64_t *hv_desc = nullptr;   // nheavy: descriptor
    const int32_t *hv_cstart = nullptr;  // nchunk + 1
    const int32_t *hv_crow = nullptr;    // nchunk
    const int32_t *hv_rowchunks = nullptr;  // nbr: chunks of each block row
    int64_t nheavy = 0, nchunk = 0;
    const uint8_t *pay = nullptr;
    // Segment-loop tasks (PULL_TASK_SEGS consecutive segments each) in
    // descending order of their stored-COO work, so that the waves, dealt
    // the tasks in this order, get even shares (NULL: the tasks in segment
    // order, as for a matrix converted on the device).
    const int32_t *task_order = nullptr;
    int32_t ntask = 0;
    // The rows that hold entries, a 16-bit mask per block row, two per word
    // ((nbr + 1) / 2 words; NULL when not known, as for a matrix converted
    // on the device).  BFS counts the other rows as reached from the start:
    // no edge leads to them, and the pull levels then skip whole block rows
    // sooner.
    const uint32_t *row_occ = nullptr;
    // Block list (valued matrices whose blocks hold at least
    // BLOCK_LIST_ENTRIES entries on average; ab_col NULL for others): every
    // block, by block row, within it by class (mfma_class), within that by
    // block column -- block column, descriptor, and where class k of block
    // row R begins at [MC_COUNT R + k] (MC_COUNT nbr + 1).  The matrix-core
    // pass for dense activations walks it.
    const int32_t *ab_col = nullptr;
    const uint64_t *ab_desc = nullptr;
    const int32_t *ab_rptr = nullptr;
    // Row-entry view (re_nchunk = 0: the matrix has none): every entry in row
    // order with ascending columns -- the column word (bit 31: first entry of
    // its row) and the value -- padded to whole chunks of RE_CHUNK entries;
    // re_row lists the rows that hold entries; re_chord[c] is the index among
    // them of the row of the entry before chunk c (-1 for the first chunk).
    // Pull streams it (k_entry_pull) when most entries sit in short COO
    // blocks, whose slot and descriptor words outweigh the entries.
    const uint32_t *re_col = nullptr;
    const void *re_val = nullptr;
    const int32_t *re_row = nullptr;
    const int32_t *re_chord = nullptr;
    int32_t re_nnz = 0, re_nchunk = 0;
    // Column-entry view (with the row-entry view): the rows and values of
    // each column's entries, column j's at ce_ptr[j] .. ce_ptr[j + 1] - 1 in
    // no fixed order.  Push walks the listed columns there (k_entry_push).
    const int32_t *ce_ptr = nullptr;  // n + 1
    const int32_t *ce_row = nullptr;
    const void *ce_val = nullptr;
    // SpMSpV runs over the entry views (most entries sit in short COO
    // blocks); a pattern matrix of filled blocks has the views for BFS only.
    bool re_sparse = false;
    // BFS, square matrices: {first entry, its column} per row and the end
    // (m + 1; a row without entries repeats the next row's first entry).
    const int2 *re_info = nullptr;
};

// Below this many entries per block the block walk of k_rows_mfma (about 70
// vector instructions a block) costs more than the pull over slots or entries.
constexpr int64_t BLOCK_LIST_ENTRIES = 8;
// Zeroed bytes behind the payload: a whole value run (MC_RUN fp32 values) read
// from the last record stays inside the allocation.
constexpr size_t PAYLOAD_PAD = 512;

// Push work items and tasks share a 64-bit count: tasks in the low bits.
constexpr int EV_TASK_BITS = 32;

// BFS over the entry views.  BfsCount: the vertices found for one level --
// items << EV_TASK_BITS | column entries of those listed as push items, the
// number of the others, whether the list is incomplete, and the nonzero
// vector blocks (kept only when the selector asks for them).  BfsRecord: what
// the host reads.
struct BfsCount {
    uint64_t items;
    uint64_t ent;         // entries of the others
    uint64_t seen, prev;  // entries of all levels before, and of the one before
    uint32_t extra, inc, nvb, pad;
};
constexpr int BFS_RECORD_LEVELS = 64;
struct BfsRecord {
    int32_t levels, reached;
    int32_t path[BFS_RECORD_LEVELS], frontier[BFS_RECORD_LEVELS];
};
// Scratch, written afresh by every BFS.
struct DevBfs {
    uint32_t *vis = nullptr, *bits[3] = {nullptr, nullptr, nullptr};
    int4 *items[2] = {nullptr, nullptr};
    BfsCount *cnt = nullptr;  // 4: three in turn, one for a list rebuilt
    BfsRecord *rec = nullptr;
};

// Segments per segment-loop task: two wave iterations of 16 segments.
constexpr int32_t PULL_TASK_SEGS = 32;

// Counter slots in the context's device counter array.
enum Counter : int {
    C_NZBLK = 0,     // nonzero vector blocks of this call
    C_TASKS = 1,     // push block tasks (sum of block-CSC lengths of active columns)
    C_PATH = 2,      // 1 push, 2 pull
    C_YNNZ = 3,      // entries written to y
    C_XBAD = 4,      // x indices out of range, counted by the blocker during this call
    C_ERR_LAST = 5,  // error bits of the last completed call
    // (6: unused)
    C_NZACC = 7,     // nonzero vector blocks, summed by the scan tiles (consumed by its last tile)
    C_NTB = 8,       // push work items (nonzero vector blocks with a nonempty block column)
    C_XPOP = 9,      // distinct x indices (mask popcounts), summed by the scan tiles
    C_SYNCERR = 10,  // single launch: a bounded wait for other workgroups ran out
    C_EITEMS = 12,   // (64 bits) push items and tasks over the column-entry view (k_entry_scatter)
    C_ECOUNT = 14,   // (64 bits) distinct x indices << 32 | nonzero vector blocks (k_entry_scatter)
    C_COUNT = 16
};
constexpr int PATH_PUSH = 1, PATH_PULL = 2;
#ifndef HV_CHUNK_BLOCKS
#define HV_CHUNK_BLOCKS 16
#endif
// blocks per chunk of the non-COO list (at most one per lane of a quarter-wave)
constexpr int HV_CHUNK = HV_CHUNK_BLOCKS;
static_assert(HV_CHUNK >= 1 && HV_CHUNK <= 16, "chunk size");

// Tile sizes of the look-back scans (vector blocks per thread of the active
// block scan; 32-row structure words per workgroup of the y compaction).
#ifndef SCAN_ITEMS_PER_THREAD
#define SCAN_ITEMS_PER_THREAD 4
#endif
#ifndef FINALIZE_WORDS
#define FINALIZE_WORDS 128
#endif
int32_t scan_tiles(int32_t nbc);      // workgroups (and status words) of the scan
int32_t finalize_tiles(int32_t nbr);  // workgroups (and status words) of the compaction

// Per-context scratch.  Every buffer is sized for the largest matrix the
// context was created for and is all-zero between calls (each call clears
// exactly what it touched).
struct DevCtx {
    void *xd = nullptr;           // dense x values, 16 * nbc entries (fp32 or fp16)
    uint32_t *xmask = nullptr;    // blk_x_mask, two 16-bit masks per word
    int32_t nxwords = 0;
    uint32_t *xbits = nullptr;    // one activity bit per vector block, written by the scan
    // push work items, one per active vector block with blocks, ascending
    // (nbc + 1): {first task (exclusive scan of block-CSC lengths), vector
    // block, pbase, 0}; task t of item a visits block-CSC position pbase + t;
    // item NT holds the task count
    int4 *items = nullptr;
    double *yacc = nullptr;       // y accumulators (16 * nbr)
    uint32_t *ybits = nullptr;    // y structure, two 16-bit row-block masks per word
    int32_t nywords = 0;
    uint32_t *visited = nullptr;  // BFS visited bitmap (row-block words)
    uint32_t *nextm = nullptr;    // BFS next-frontier bitmap
    int32_t *counters = nullptr;  // C_COUNT int32
    int32_t *rdone = nullptr;     // nbr: chunks of a block row committed so far (dense-output pass)
    // Look-back status words of the two scans, in two copies each: a call
    // uses copy `parity` and clears the other copy for the next call, so no
    // other kernel has to clean up after a scan.
    uint64_t *st_scan[2] = {nullptr, nullptr};  // active-block scan
    int32_t n_st_scan = 0;
    uint64_t *st_fin[2] = {nullptr, nullptr};   // y compaction
    int32_t n_st_fin = 0;
    int scan_parity = 0, fin_parity = 0;
    // Compacted pull (moderate x activity): per-wave regions of active slot
    // ids and their counts; written and read within one call.
    int32_t *clist = nullptr;
    int64_t clist_cap = 0;
    uint32_t *ccount = nullptr;
    // Single launch (short index lists): ready / all-done words (eight
    // copies) and one done word per workgroup (SYNC_WORDS in all), and the
    // number of the last such call (the words hold it once written; 0 is
    // never used).
    uint32_t *sync = nullptr;
    uint32_t gen = 0;
};
constexpr int32_t SYNC_WORDS = 8 * 1024 + 4096;
// Entries and regions of the compacted pull's list for a matrix of nseg
// pull segments.
int64_t compact_list_entries(int64_t nseg);
int32_t compact_list_regions();

enum Mode : int { M_F32 = 0, M_F16 = 1, M_BOOL = 2, M_BFS = 3 };

// Workgroups of `kernel` (threads wide, dyn_lds bytes of dynamic LDS) that the
// current device holds at once, or 0 if it cannot be asked.  Any thread may
// call it; answers are kept per device, kernel and LDS size.
int resident_workgroups(const void *kernel, int threads, size_t dyn_lds);
hipError_t launch_scatter(const DevMatrix &A, const DevCtx &C, int mode, int32_t k,
                          const int32_t *x_idx, const void *x_val, hipStream_t s);
hipError_t launch_ballot(const DevMatrix &A, const DevCtx &C, int mode, const void *x_dense,
                         hipStream_t s);
// th3s > 0: the spread rule as well; tasks_max >= 0: push iff fewer push
// tasks than that, in place of both (BFS levels; see k_scan)
hipError_t launch_scan(const DevMatrix &A, DevCtx &C, int forced_path, double th3, double th3s,
                       hipStream_t s, double tasks_max = -1.0);
// Blocker and scan as one single-workgroup kernel, for up to SMALL_X_MAX
// indices and an activity bitmap of up to SMALL_X_WORDS words (small_x_fits);
// otherwise launch_scatter + launch_scan.
constexpr int32_t SMALL_X_MAX = 2048;
constexpr int32_t SMALL_X_WORDS = 8192;
bool small_x_fits(const DevMatrix &A, int32_t k);
hipError_t launch_small_x(const DevMatrix &A, const DevCtx &C, int mode, int32_t k, const int32_t *x_idx,
                          const void *x_val, int forced_path, double th3, double th3s, hipStream_t s);
// Blocker, selector, traversal and compaction of y in one launch, for an
// index list small_x_fits accepts whose activity bitmap also fits the pull
// kernel's LDS copy (fused_fits); valued and OR-AND modes.
bool fused_fits(const DevMatrix &A, int32_t k);
hipError_t launch_fused(const DevMatrix &A, DevCtx &C, int mode, int32_t k, const int32_t *x_idx,
                        const void *x_val, const uint32_t *omask, int complement, int forced_path, double th3,
                        double th3s, int32_t *y_idx, void *y_val, int32_t *y_nnz, hipStream_t s);
// Dense activation with n a multiple of 16 and a 16-byte aligned x: the
// blocker runs inside the scan (one launch fewer).
bool scan_takes_dense(const DevMatrix &A, const void *x_dense);
hipError_t launch_scan_dense(const DevMatrix &A, DevCtx &C, int mode, const void *x_dense, int forced_path,
                             double th3, double th3s, hipStream_t s);
// Launches the traversal: the pull kernel then the push kernel for an
// automatic path (the one the scan did not choose returns at once; the push
// kernel also walks the compacted pull's list), or only what the forced path
// needs.
hipError_t launch_main(const DevMatrix &A, const DevCtx &C, int mode, const void *xd,
                       const uint32_t *omask, int complement, int32_t *parent, int forced_path,
                       hipStream_t s);
// Traversals over the entry views (A.re_nchunk > 0), any mode but BFS.  The
// blocker counts in C_XBAD, C_EITEMS and (count) C_ECOUNT, which the
// compaction of y clears; the traversals write no counter.
//   launch_entry_scatter  blocker that also lists push items (into C.items:
//                         at most one per x index), as push and auto need;
//                         count: and counts what the automatic choice asks for
//   launch_entry_pull     pull; scanned: a scan ran, and the kernel returns
//                         at once when its choice is push; dense_out: the y
//                         structure is not wanted
//   launch_entry_push     push
//   launch_entry_auto     the choice is taken on the device
//   entry_pull_pays       whether pull with a sparse x over the views is the
//                         faster way
bool entry_pull_pays(const DevMatrix &A, int mode);
hipError_t launch_entry_scatter(const DevMatrix &A, const DevCtx &C, int mode, int32_t k, const int32_t *x_idx,
                                const void *x_val, bool count, hipStream_t s);
hipError_t launch_entry_pull(const DevMatrix &A, const DevCtx &C, int mode, const uint32_t *omask, int complement,
                             bool scanned, bool dense_out, hipStream_t s);
hipError_t launch_entry_push(const DevMatrix &A, const DevCtx &C, int mode, const uint32_t *omask, int complement,
                             hipStream_t s);
hipError_t launch_entry_auto(const DevMatrix &A, const DevCtx &C, int mode, const uint32_t *omask, int complement,
                             double th3, double th3s, hipStream_t s);
// Column-entry view from the row-entry view: entries per column (cnt zeroed
// before), then their rows and values at next[column]++ (vb value bytes).
hipError_t launch_ce_count(const DevMatrix &A, int32_t *cnt, hipStream_t s);
hipError_t launch_ce_fill(const DevMatrix &A, int32_t vb, int32_t *next, int32_t *ce_row, void *ce_val, hipStream_t s);
hipError_t launch_finalize(const DevMatrix &A, DevCtx &C, int mode, int32_t *y_idx,
                           void *y_val, int32_t *y_nnz, const int32_t *x_idx, int32_t k,
                           hipStream_t s);
hipError_t launch_finalize_dense(const DevMatrix &A, const DevCtx &C, int mode, void *y,
                                 float *y32, hipStream_t s);
// Dense activation, pull on a matrix without COO blocks: the non-COO pass
// reading the activation itself, with no scan before it and writing the
// dense output y (and y32 when not NULL) itself (k_rows_dx), when
// rows_dx_fits (for a valued matrix: the conditions of scan_takes_dense, no
// COO block, at most ROWS_DX_MAX_NBC vector blocks).
bool rows_dx_fits(const DevMatrix &A, const void *x_dense);
hipError_t launch_rows_dx(const DevMatrix &A, const DevCtx &C, int mode, const void *x_dense, void *y,
                          float *y32, hipStream_t s);
// Dense activations (1 <= nb <= 8, rows of x) on a matrix with a block list
// (rows_mfma_fits), in one kernel on the matrix cores.  With rows_mfma_parts
// > 1 it sums through yacc (nb sets of 16 nbr accumulators, zero between
// calls) and the context's block-row counts; else it touches no scratch.
bool rows_mfma_fits(const DevMatrix &A);
int32_t rows_mfma_parts(const DevMatrix &A);
hipError_t launch_rows_mfma(const DevMatrix &A, const DevCtx &C, double *yacc, int32_t nb, const void *x, void *y,
                            float *y32, hipStream_t s);
// Batched dense activations (NB in {2, 4, 8} vectors per pass, nb <= NB of
// them real): the padded copies into xdb (NB * 16 nbc entries) and their
// union mask; the pull over a matrix without COO blocks into yaccb (NB * 16
// nbr accumulators); the dense outputs of the nb real vectors.
hipError_t launch_ballot_batch(const DevMatrix &A, const DevCtx &C, int mode, const void *x, int32_t nb,
                               int32_t NB, void *xdb, hipStream_t s);
hipError_t launch_rows_batch(const DevMatrix &A, const DevCtx &C, int mode, int32_t NB, const void *xdb,
                             double *yaccb, hipStream_t s);
hipError_t launch_finalize_batch(const DevMatrix &A, const DevCtx &C, int mode, int32_t nb, int32_t NB,
                                 double *yaccb, void *y, float *y32, hipStream_t s);
// BFS over the entry views (A.re_info): the start, then one launch per level;
// a level after the last returns at once.  policy 0 with th3 <= 0 pushes by
// the rule at DBS_BFS_PUSH_ENTRIES, push_share being that share.
hipError_t launch_bfs_start(const DevMatrix &A, const DevBfs &B, int32_t source, int32_t *level, int32_t *parent,
                            hipStream_t s);
hipError_t launch_bfs_level(const DevMatrix &A, const DevBfs &B, int32_t l, int32_t *level, int32_t *parent,
                            int policy, double th3, double push_share, hipStream_t s);
hipError_t launch_bfs_init(const DevMatrix &A, const DevCtx &C, int32_t source, int32_t *level,
                           int32_t *parent, hipStream_t s);
hipError_t launch_bfs_update(const DevMatrix &A, const DevCtx &C, int32_t next_level,
                             int32_t *level, hipStream_t s);
hipError_t launch_bfs_finish(const DevMatrix &A, int32_t *parent, hipStream_t s);


}  // namespace dbs
