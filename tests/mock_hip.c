/* A stand-in for the parts of the HIP runtime that the library calls, preloaded in
 * front of it: memory is host memory, launches are recorded by kernel name and run
 * nothing. Allocations larger than a limit fail. For tests of host code on the CPU. */
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
static size_t limit = (size_t)-1, largest, total;
static int allocations, failures;
static char log_[1 << 16];
static struct { const void *host; const char *name; } kernels[1024];
static int nkernels;

void mock_reset(size_t max_bytes) { limit = max_bytes; largest = total = 0; allocations = failures = 0; log_[0] = 0; }
const char *mock_log(void) { return log_; }
size_t mock_largest(void) { return largest; }
int mock_allocations(void) { return allocations; }
int mock_failures(void) { return failures; }

static void note(const char *name)
{
    if (strlen(log_) + strlen(name) + 2 < sizeof log_) { strcat(log_, name); strcat(log_, "\n"); }
}

void __hipRegisterFunction(void *m, const void *host, char *dev, const char *name, unsigned t, void *a, void *b, void *c, void *d, int *w)
{
    (void)m; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (nkernels < 1024) { kernels[nkernels].host = host; kernels[nkernels++].name = strdup(name); }
}

static int get(void **p, size_t n)
{
    if (n > limit) { ++failures; *p = NULL; return 2; }   /* hipErrorOutOfMemory */
    ++allocations;
    total += n;
    if (n > largest) largest = n;
    return posix_memalign(p, 256, n ? n : 1) ? 2 : 0;
}

int hipMalloc(void **p, size_t n) { return get(p, n); }
int hipMallocAsync(void **p, size_t n, void *st) { (void)st; return get(p, n); }
int hipFree(void *p) { free(p); return 0; }
int hipFreeAsync(void *p, void *st) { (void)st; free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipMemGetAddressRange(void **b, size_t *n, void *p) { (void)p; *b = NULL; *n = (size_t)-1; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; static char array[64]; *p = array; return 0; }
int hipModuleLoadData(void **m, const void *i) { (void)i; *m = (void *)1; note("module"); return 0; }
int hipModuleGetFunction(void **f, void *m, const char *n) { (void)m; (void)n; *f = (void *)1; return 0; }
int hipModuleUnload(void *m) { (void)m; return 0; }
int hipModuleLaunchKernel(void *f, unsigned a, unsigned b, unsigned c, unsigned d, unsigned e, unsigned g, unsigned l, void *st, void **p, void **x)
{
    (void)f; (void)a; (void)b; (void)c; (void)d; (void)e; (void)g; (void)l; (void)st; (void)p; (void)x;
    note("generated");
    return 0;
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void *st) { (void)g; (void)b; (void)l; (void)st; return 0; }
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *l, void **st)
{
    memset(g, 0, sizeof *g);
    memset(b, 0, sizeof *b);
    *l = 0;
    *st = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **a, size_t l, void *st)
{
    (void)g; (void)b; (void)a; (void)l; (void)st;
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].host == f) { note(kernels[i].name); return 0; }
    note("?");
    return 0;
}
