/* Stand-in for the HIP runtime calls of libpic's host code, preloaded by tests
 * that run without a GPU: nothing is executed, "device" memory is addresses
 * only.  It records the device range that copies and fills reach, and the
 * graphs that are alive, and can fail the n-th instantiation.  A copy to the host
 * gives zeros, or a word that the test sets. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

uint64_t stub_lo, stub_hi;          /* device addresses that may be written */
uint64_t stub_outside;              /* fills and copies that left them */
int64_t stub_word;                  /* what an 8-byte copy to the host gives */
int stub_graphs, stub_execs;        /* alive */
int stub_fail_instantiate;          /* 1-based count of the call that fails, 0: none */
static int instantiated;

static void touch(void *p, size_t n)
{
    const uint64_t a = (uint64_t)p;
    if (stub_hi && n && (a < stub_lo || a + n > stub_hi)) ++stub_outside;
}
static int copy(void *d, const void *s, size_t n, int kind)
{
    (void)s;
    if (kind == 1) touch(d, n);             /* host to device */
    else if (kind == 2) {                   /* device to host: zeros, or the word set */
        memset(d, 0, n);
        if (n == sizeof(stub_word)) memcpy(d, &stub_word, n);
    }
    return 0;
}

int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "stub"; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)((uint64_t)1 << 44); return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l)
{
    (void)f; (void)b; (void)l;
    *n = 2;
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return copy(d, s, n, kind); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)st; return copy(d, s, n, kind); }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)v; (void)st; touch(d, n); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)1; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return 0; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = (void *)2; ++stub_graphs; return 0; }
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t z)
{
    (void)g; (void)n; (void)l; (void)z;
    if (++instantiated == stub_fail_instantiate) return 1;
    *e = (void *)3;
    ++stub_execs;
    return 0;
}
int hipGraphDestroy(void *g) { (void)g; --stub_graphs; return 0; }
int hipGraphExecDestroy(void *e) { (void)e; --stub_execs; return 0; }
int hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventCreate(void **e) { *e = (void *)4; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return 0; }
typedef struct { unsigned x, y, z; } dim3_;
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **a, size_t l, void *s)
{
    (void)f; (void)g; (void)b; (void)a; (void)l; (void)s;
    return 0;
}
