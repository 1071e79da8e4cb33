/* Host stand-ins for the HIP functions that the library calls, for tests of
 * its host side without a GPU: "device" memory is host memory, kernels are
 * not run, and allocations can be made to fail.  Loaded with RTLD_GLOBAL
 * before the library, whose calls then bind here. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

typedef int err_t; /* hipError_t: 0 success, 1 invalid value, 2 out of memory */
typedef struct {
    uint32_t x, y, z;
} dim_t;

long fake_allocs, fake_frees, fake_host_allocs, fake_fail_at = -1, fake_fail_from = -1, fake_occupancy_calls, fake_launches;
int fake_device, fake_cus = 256, fake_per_cu = 1;
static __thread uint32_t last_grid; /* of this thread's last kernel with dynamic LDS: a traversal */
static __thread err_t last_error; /* stays until it is read, as the runtime's */

static err_t done(err_t e)
{
    if (e) last_error = e;
    return e;
}
static err_t get(void **p, size_t n)
{
    const long k = __sync_fetch_and_add(&fake_allocs, 1);
    if (k == fake_fail_at || (fake_fail_from >= 0 && k >= fake_fail_from)) {
        *p = NULL;
        return done(2);
    }
    *p = calloc(n ? n : 1, 1);
    return done(*p ? 0 : 2);
}
err_t hipMalloc(void **p, size_t n) { return get(p, n); }
err_t hipFree(void *p)
{
    if (p) __sync_fetch_and_add(&fake_frees, 1);
    free(p);
    return 0;
}
err_t hipHostMalloc(void **p, size_t n, unsigned f)
{
    (void)f;
    __sync_fetch_and_add(&fake_host_allocs, 1);
    *p = calloc(n ? n : 1, 1);
    return done(*p ? 0 : 2);
}
err_t hipHostFree(void *p)
{
    free(p);
    return 0;
}
err_t hipMemcpy(void *d, const void *s, size_t n, int k)
{
    (void)k;
    if (n) memcpy(d, s, n);
    return 0;
}
err_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st)
{
    (void)st;
    return hipMemcpy(d, s, n, k);
}
err_t hipMemset(void *d, int v, size_t n)
{
    memset(d, v, n);
    return 0;
}
err_t hipMemsetAsync(void *d, int v, size_t n, void *st)
{
    (void)st;
    return hipMemset(d, v, n);
}
err_t hipStreamSynchronize(void *s)
{
    (void)s;
    return 0;
}
err_t hipGetDevice(int *d)
{
    *d = fake_device;
    return 0;
}
err_t hipGetDeviceCount(int *n)
{
    *n = 2;
    return 0;
}
err_t hipDeviceGetAttribute(int *v, int a, int d)
{
    (void)a;
    *v = fake_cus / (d + 1); /* device 1 has half of the compute units */
    return 0;
}
err_t hipGetDevicePropertiesR0600(void *prop, int d)
{
    extern const size_t fake_arch_offset, fake_prop_bytes;
    (void)d;
    memset(prop, 0, fake_prop_bytes);
    strcpy((char *)prop + fake_arch_offset, "gfx950");
    return 0;
}
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int t, size_t lds)
{
    (void)f;
    (void)t;
    (void)lds;
    __sync_fetch_and_add(&fake_occupancy_calls, 1);
    usleep(200);
    *n = fake_per_cu;
    return 0;
}
err_t hipGetLastError(void)
{
    const err_t e = last_error;
    last_error = 0;
    return e;
}
const char *hipGetErrorString(err_t e) { return e == 2 ? "out of memory" : "error"; }
err_t hipGetSymbolAddress(void **p, const void *s)
{
    (void)s;
    *p = NULL;
    return done(1);
}
err_t hipEventCreate(void **e)
{
    *e = NULL;
    return done(1);
}
err_t hipEventDestroy(void *e)
{
    (void)e;
    return 0;
}
err_t hipEventRecord(void *e, void *s)
{
    (void)e;
    (void)s;
    return 0;
}
err_t hipEventElapsedTime(float *ms, void *a, void *b)
{
    (void)a;
    (void)b;
    *ms = 0;
    return 0;
}
uint32_t fake_grid(void) { return last_grid; }
static __thread struct {
    dim_t grid, block;
    size_t lds;
    void *stream;
} call;
err_t __hipPushCallConfiguration(dim_t g, dim_t b, size_t lds, void *s)
{
    call.grid = g;
    call.block = b;
    call.lds = lds;
    call.stream = s;
    return 0;
}
err_t __hipPopCallConfiguration(dim_t *g, dim_t *b, size_t *lds, void **s)
{
    *g = call.grid;
    *b = call.block;
    *lds = call.lds;
    *s = call.stream;
    return 0;
}
/* this library's kernels by host function, and the names of those launched, in order */
static struct {
    const void *f;
    const char *name;
} kernels[1024];
static int nkernels;
static __thread char launched[1 << 12];
const char *fake_launched(void) { return launched; }
void fake_forget(void) { launched[0] = 0; }
err_t hipLaunchKernel(const void *f, dim_t g, dim_t b, void **args, size_t lds, void *s)
{
    const size_t at = strlen(launched);
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].f == f && at + strlen(kernels[i].name) + 2 < sizeof launched) {
            strcpy(launched + at, kernels[i].name);
            strcat(launched, " ");
        }
    (void)args;
    (void)s;
    __sync_fetch_and_add(&fake_launches, 1);
    if (lds) last_grid = g.x;
    return b.x && g.x ? 0 : done(1);
}
void **__hipRegisterFatBinary(const void *d)
{
    static void *h;
    (void)d;
    return &h;
}
void __hipRegisterFunction(void **m, const void *h, char *n, const char *d, unsigned t, void *a, void *b, void *c, void *e, int *w)
{
    if (strstr(d, "3dbs") && nkernels < 1024) {
        kernels[nkernels].f = h;
        kernels[nkernels++].name = strdup(d);
    }
    (void)m, (void)n, (void)t, (void)a, (void)b, (void)c, (void)e, (void)w;
}
void __hipRegisterVar(void **m, void *v, char *h, char *n, int e, size_t s, int c, int g)
{
    (void)m, (void)v, (void)h, (void)n, (void)e, (void)s, (void)c, (void)g;
}
void __hipUnregisterFatBinary(void **m) { (void)m; }
