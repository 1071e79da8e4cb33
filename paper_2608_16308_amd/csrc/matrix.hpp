// The device-resident matrix object of the C ABI, shared by the upload path
// (api.hip) and the GPU-side conversion (convert.hip).
#pragma once
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"

struct dbs_matrix {
    dbs::DevMatrix d;
    dbs_matrix_info info{};
    std::vector<void *> allocs;  // device allocations owned by the matrix
};

// Reports a failed HIP call.  The runtime keeps the error until it is asked for
// it, and every launch here asks: it is taken back, so that no later launch
// reports it.
inline thread_local bool g_out_of_memory = false;  // (of the last one on this thread)
inline dbs_status hip_fail(hipError_t e, const char *what)
{
    (void)hipGetLastError();
    g_out_of_memory = e == hipErrorOutOfMemory;
    return dbs_fail(DBS_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

// Whether `st` reports that memory ran out, on the host or on the device.
inline bool out_of_memory(dbs_status st)
{
    return st == DBS_ERR_ALLOC || (st == DBS_ERR_DEVICE && g_out_of_memory);
}

// Adds arrays that a matrix can do without (entry views, the block list: every
// call has a way over the blocks): make() allocates into A->allocs and sets
// their fields in A->d.  Without memory for them the matrix is as it was.
template <class Make>
dbs_status optional_arrays(dbs_matrix *A, Make &&make)
{
    const size_t had = A->allocs.size();
    const dbs::DevMatrix before = A->d;
    const dbs_status st = make();
    if (!out_of_memory(st)) return st;
    for (size_t i = had; i < A->allocs.size(); ++i) (void)hipFree(A->allocs[i]);
    A->allocs.resize(had);
    A->d = before;
    return DBS_OK;
}

// Adds the column-entry view of a matrix that has its row-entry view (on the
// default stream; returns when done).
dbs_status column_entries(dbs_matrix *A);
