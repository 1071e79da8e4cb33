// Builds a matrix with every single host allocation failing in turn: the
// build either reports DBS_ERR_ALLOC or succeeds (a failed entry view is left
// out, a thread that cannot be started done without), never ends the process,
// and what it built is the same.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

static std::atomic<long> g_count{0}, g_fail_at{-1};
static std::atomic<bool> g_from{false};  // fail from there on
static void *take(size_t n)
{
    const long k = g_count.fetch_add(1), f = g_fail_at;
    if (f >= 0 && (k == f || (g_from && k > f))) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(size_t n) { return take(n); }
void *operator new[](size_t n) { return take(n); }
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
    try {
        return take(n);
    } catch (...) {
        return nullptr;
    }
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }

#include "../../paper_2608_16308_amd/csrc/builder.cpp"

int main()
{
    setenv("DBS_BUILD_THREADS", "3", 1);
    // rows of four entries far apart, columns not in order
    const int32_t m = 9000, n = 9000;
    std::vector<int64_t> rp((size_t)m + 1);
    std::vector<int32_t> ci;
    std::vector<float> v;
    for (int32_t i = 0; i < m; ++i) {
        for (int32_t k : {3, 0, 2, 1}) {
            ci.push_back((k * 2250 + (i * 17) % 2250) % n);
            v.push_back((float)(i + k) + 0.5f);
        }
        rp[(size_t)i + 1] = (int64_t)ci.size();
    }
    auto build = [&](dbs_host_matrix **h) {
        return dbs_host_build_csr(m, n, (int64_t)ci.size(), rp.data(), ci.data(), v.data(), DBS_F32, nullptr, h);
    };
    dbs_host_matrix *want = nullptr;
    if (build(&want) != DBS_OK || want->nre_chunk == 0) return std::printf("no reference build\n"), 1;
    long ok = 0, refused = 0, without = 0, bad = 0;
    for (int from = 0; from < 2; ++from) {
        for (long k = 0;; ++k) {
            dbs_host_matrix *h = nullptr;
            g_from = from != 0;
            g_count = 0;
            g_fail_at = k;
            const dbs_status st = build(&h);
            g_fail_at = -1;
            const bool reached = g_count > k;
            if (st == DBS_OK) {
                ++ok;
                if (h->nre_chunk == 0) ++without;
                if (h->nre_chunk == 0 && (h->re_col || h->re_val || !h->re_row.empty() || !h->re_info.empty())) ++bad;
                if (h->nre_chunk > 0 && (h->re_row != want->re_row || h->re_chord != want->re_chord ||
                                         std::memcmp(h->re_col.get(), want->re_col.get(), (size_t)h->nre_chunk * RE_CHUNK * 4)))
                    ++bad;
                if (h->payload != want->payload || h->desc != want->desc || h->csc2csr != want->csc2csr) ++bad;
            } else {
                ++refused;
                if (st != DBS_ERR_ALLOC || h) ++bad;
            }
            dbs_host_destroy(h);
            if (!reached) break;
        }
    }
    dbs_host_destroy(want);
    std::printf("%ld built, %ld of them without the entry view, %ld refused, %ld wrong\n", ok, without, refused, bad);
    return bad || !without || !refused ? 1 : 0;
}
