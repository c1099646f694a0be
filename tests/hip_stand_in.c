/* Stand-in for the HIP runtime calls that libnavsim.so makes, for tests of its
 * host code without a GPU: device memory is host memory, a launch is only
 * recorded (by kernel name), and every call is counted.  Loaded with global
 * symbols before the library, its definitions take the runtime's place.
 * Allocations can be told to fail, and a stream capture in progress (in the
 * global mode) can be declared: calls that HIP forbids then fail, unless the
 * thread has put itself in the relaxed mode. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, INVALID = 1, OOM = 2, CAPTURE = 900 };
enum { MAX_KERNELS = 1 << 16, MAX_LAUNCHES = 4096, SCRATCH = 16 << 20 };

static struct { const void *f; const char *name; } kernels[MAX_KERNELS];
static int n_kernels;
static const char *launches[MAX_LAUNCHES];
static int n_launches, n_malloc, n_free, n_sync, n_copy, fail_malloc = -1, fail_one = -1, capturing, mode;
static unsigned char *scratch;
static int n_scratch; /* pointers into it among the proposal launches' arguments */

/* --- read and set by the tests --- */
int stand_in_scratch_pointers(void) { return n_scratch; }
void stand_in_clear(void) { n_scratch = n_launches = n_malloc = n_free = n_sync = n_copy = 0; }
void stand_in_counts(int *o) {
    o[0] = n_launches;
    o[1] = n_malloc;
    o[2] = n_free;
    o[3] = n_sync;
    o[4] = n_copy;
}
const char *stand_in_launch(int i) { return i < n_launches && i < MAX_LAUNCHES ? launches[i] : ""; }
const char *stand_in_kernel(int i) { return i < n_kernels ? kernels[i].name : ""; } /* compiled in */
void stand_in_fail_malloc(int after) { fail_malloc = after; }    /* that many succeed; -1: all */
void stand_in_fail_one_malloc(int after) { fail_one = after; }  /* only the one after that many */
void stand_in_capturing(int on) { capturing = on; }

static int forbidden(void) { return capturing && mode == 0; }

/* --- the runtime --- */
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipSetDevice(int d) { return d == 0 ? OK : 101; }
int hipGetDeviceCount(int *n) { *n = 1; return OK; }
int hipDeviceGetAttribute(int *v, int attr, int dev) {
    (void)dev;
    /* hipDeviceAttributeMultiprocessorCount, MaxSharedMemoryPerBlock and
       MaxSharedMemoryPerMultiprocessor in hip_runtime_api.h */
    *v = attr == 63 ? 256 : attr == 74 || attr == 10002 ? 163840 : 0;
    return OK;
}
int hipMalloc(void **p, size_t n) {
    ++n_malloc;
    *p = NULL;
    if (forbidden()) return CAPTURE;
    if (fail_one >= 0 && fail_one-- == 0) return OOM;
    if (fail_malloc == 0) return OOM;
    if (fail_malloc > 0) --fail_malloc;
    *p = malloc(n ? n : 1);
    return *p ? OK : OOM;
}
int hipFree(void *p) {
    ++n_free;
    if (forbidden()) return CAPTURE;
    free(p);
    return OK;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) {
    (void)kind;
    ++n_copy;
    if (capturing) return CAPTURE; /* the null stream waits for the capturing one */
    memcpy(d, s, n);
    return OK;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream) {
    (void)kind;
    (void)stream;
    ++n_copy;
    memcpy(d, s, n);
    return OK;
}
int hipMemset(void *d, int v, size_t n) {
    if (capturing) return CAPTURE;
    memset(d, v, n);
    return OK;
}
int hipDeviceSynchronize(void) { ++n_sync; return capturing ? CAPTURE : OK; }
int hipStreamSynchronize(void *s) { (void)s; return forbidden() ? CAPTURE : OK; }
int hipThreadExchangeStreamCaptureMode(int *m) {
    const int old = mode;
    mode = *m;
    *m = old;
    return OK;
}
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return OK; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipGetLastError(void) { return OK; }
const char *hipGetErrorString(int e) { return e == OOM ? "out of memory" : e == CAPTURE ? "stream is capturing" : "error"; }
/* hipFuncAttributes: 56 bytes, no static LDS */
int hipFuncGetAttributes(void *a, const void *f) { (void)f; memset(a, 0, 56); return OK; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int threads, size_t lds) {
    (void)f;
    const int by_waves = 16 * 64 / threads, by_lds = lds ? (int)(163840 / lds) : by_waves;
    *n = by_waves < by_lds ? by_waves : by_lds;
    return OK;
}
int hipGetSymbolAddress(void **p, const void *sym) {
    (void)sym;
    if (!scratch) scratch = calloc(1, SCRATCH);
    *p = scratch;
    return OK;
}
static dim3 c_grid, c_block;
static size_t c_lds;
static void *c_stream;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *s) {
    c_grid = g;
    c_block = b;
    c_lds = lds;
    c_stream = s;
    return OK;
}
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **s) {
    *g = c_grid;
    *b = c_block;
    *lds = c_lds;
    *s = c_stream;
    return OK;
}
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
    (void)g;
    (void)b;
    (void)lds;
    (void)s;
    const char *name = "?";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].f == f) name = kernels[i].name;
    if (strstr(name, "propose"))
        for (int i = 0; i < 19; ++i) { /* ProposeArgs: 152 bytes */
            unsigned char *p;
            memcpy(&p, (char *)args[1] + 8 * i, 8);
            n_scratch += scratch && p >= scratch && p < scratch + SCRATCH;
        }
    if (n_launches < MAX_LAUNCHES) launches[n_launches] = name;
    ++n_launches;
    return OK;
}
void **__hipRegisterFatBinary(const void *data) { (void)data; static void *m; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned limit,
                           void *tid, void *bid, dim3 *bd, dim3 *gd, int *ws) {
    (void)m; (void)dev; (void)limit; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (n_kernels < MAX_KERNELS) {
        kernels[n_kernels].f = host;
        kernels[n_kernels++].name = name;
    }
}
void __hipRegisterVar(void **m, void *var, char *host, char *dev, int ext, size_t size, int c, int g) {
    (void)m; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)c; (void)g;
}
