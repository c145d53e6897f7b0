/* Stand-in for the HIP runtime calls of libfrdvm on a machine without a GPU:
 * "device" memory is host memory, kernels are counted and not run.  Loaded
 * with RTLD_GLOBAL before the library, so that its calls resolve here.
 * Set-up (meshes, tables, buffers, error paths) then runs as it is. */
#include <stdlib.h>
#include <string.h>

typedef int hipError_t; /* 0: success, 2: out of memory */
#define MAX_ALLOC 4096
static struct { void *p; size_t n; } tab[MAX_ALLOC];
static long n_alloc, n_launch, fail_at = -1;
static size_t live_bytes, capacity = (size_t)-1;
static hipError_t last;

/* controls for the tests */
void stub_fail_at(long k) { fail_at = k; n_alloc = 0; } /* the k-th allocation from here fails (-1: none) */
void stub_capacity(size_t b) { capacity = b; }
long stub_allocs(void) { return n_alloc; }
long stub_launches(void) { return n_launch; }
size_t stub_live(void) { return live_bytes; }
void *stub_find(size_t bytes, int idx) {
    for (int i = 0; i < MAX_ALLOC; ++i)
        if (tab[i].p && tab[i].n == bytes && idx-- == 0) return tab[i].p;
    return NULL;
}

hipError_t hipMalloc(void **p, size_t n) {
    *p = NULL;
    if (n_alloc++ == fail_at || live_bytes + n > capacity) return last = 2;
    for (int i = 0; i < MAX_ALLOC; ++i)
        if (!tab[i].p) {
            *p = tab[i].p = calloc(n ? n : 1, 1);
            tab[i].n = n;
            live_bytes += n;
            return 0;
        }
    return last = 2;
}
hipError_t hipFree(void *p) {
    for (int i = 0; p && i < MAX_ALLOC; ++i)
        if (tab[i].p == p) {
            live_bytes -= tab[i].n;
            free(p);
            tab[i].p = NULL;
            return 0;
        }
    if (p) abort(); /* freed twice */
    return 0;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return 0; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return 0; }
hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
hipError_t hipGetLastError(void) { hipError_t e = last; last = 0; return e; }
const char *hipGetErrorString(hipError_t e) { (void)e; return "stub"; }
hipError_t hipDeviceSynchronize(void) { return 0; }
hipError_t hipStreamSynchronize(void *s) { (void)s; return 0; }
hipError_t hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)1; return 0; }
hipError_t hipStreamDestroy(void *s) { (void)s; return 0; }
hipError_t hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
hipError_t hipEventCreate(void **e) { *e = (void *)1; return 0; }
hipError_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = (void *)1; return 0; }
hipError_t hipEventDestroy(void *e) { (void)e; return 0; }
hipError_t hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
hipError_t hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 0; return 0; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = NULL; return 1; }

typedef struct { unsigned x, y, z; } dim3_;
hipError_t hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **a, size_t m, void *s) {
    (void)f; (void)g; (void)b; (void)a; (void)m; (void)s;
    ++n_launch;
    return 0;
}
static dim3_ cg, cb;
static size_t cm;
static void *cs;
hipError_t __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t m, void *s) { cg = g; cb = b; cm = m; cs = s; return 0; }
hipError_t __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *m, void **s) { *g = cg; *b = cb; *m = cm; *s = cs; return 0; }
