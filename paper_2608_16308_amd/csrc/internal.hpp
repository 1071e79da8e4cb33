// Host-side internals shared by the builder and the C-ABI implementation.
#pragma once
#include <cstdarg>
#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "../../include/dbspmspv.h"
#include "db_format.hpp"

// Thread-local message for dbs_last_error().
dbs_status dbs_fail(dbs_status st, const char *fmt, ...);

struct dbs_host_matrix {
    int32_t m = 0, n = 0;
    int64_t nnz = 0;
    dbs_dtype dtype = DBS_F32;
    dbs_build_opts opts{};
    int32_t nbr = 0, nbc = 0;
    int64_t nblk = 0, nseg = 0;
    int64_t by_type[DBS_NUM_BLOCK_TYPES] = {0, 0, 0, 0, 0};
    std::vector<int32_t> rb_ptr;   // nbr + 1
    std::vector<int32_t> cb_col;   // nblk
    std::vector<int32_t> cb_ptr;   // nbc + 1
    std::vector<int32_t> csc_row;  // nblk
    std::vector<int32_t> csc2csr;  // nblk
    std::vector<uint64_t> desc;    // nblk
    std::vector<uint64_t> seg;     // nseg
    // (nbr + 1) / 2 words, a 16-bit mask per block row (two per word): the
    // rows that hold at least one entry
    std::vector<uint32_t> row_occ;
    std::vector<uint8_t> payload;
    // Row-entry view (see DevMatrix; empty when the matrix has none): the
    // entries in row order with ascending columns.
    std::unique_ptr<uint32_t[]> re_col;  // nre_chunk * RE_CHUNK words
    std::unique_ptr<uint8_t[]> re_val;   // nnz values (NULL for a pattern)
    std::vector<int32_t> re_row, re_chord;
    std::vector<uint64_t> re_info;       // square matrices: first entry | its column << 32
    bool re_sparse = false;
    int64_t nre_chunk = 0;
};

inline uint32_t dtype_bytes(dbs_dtype t) { return t == DBS_F32 ? 4u : (t == DBS_F16 ? 2u : 0u); }

// Whether SpMSpV runs over the entry views: the matrix is a list of short COO
// blocks more than one of filled blocks (at least half of its entries sit in
// COO blocks) and was not asked to hold one block format.
inline bool entries_sparse(int64_t nnz, int64_t coo_entries, int32_t force_type)
{
    return 2 * coo_entries >= nnz && force_type < 0;
}
// Whether a matrix gets entry views (entry positions fit 32 bits): for
// SpMSpV, or, a pattern, for BFS.
inline bool entries_wanted(int64_t nnz, bool sparse, int32_t dtype, int32_t force_type)
{
    return nnz > 0 && nnz <= (int64_t)INT32_MAX - dbs::RE_CHUNK && (sparse || (dtype == DBS_PATTERN && force_type < 0));
}

void fill_info(const dbs_host_matrix &h, dbs_matrix_info *out);
