/* A stand-in for the HIP runtime that launches nothing and records every
 * launch: the tests load it in front of libccl.so, in a process of its own, to
 * see which kernels a call would launch and with which grids, for any size and
 * without a GPU.  Like HIP it refuses a grid of 2^32 threads or more in x. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } Dim3;

enum { kMaxKernels = 1024, kMaxLaunches = 4096, kInvalidConfiguration = 9 };
static struct { const void *fn; const char *name; } g_kernel[kMaxKernels];
static int g_kernels;
static struct { const char *name; Dim3 grid, block; int refused; } g_launch[kMaxLaunches];
static int g_launches, g_last;
static struct { Dim3 grid, block; size_t shared; void *stream; } g_config;
static char g_heap[1 << 12];

/* read by the tests */
int rec_count(void) { return g_launches; }
const char *rec_name(int i) { return g_launch[i].name; }
void rec_get(int i, uint32_t *v) {
    v[0] = g_launch[i].grid.x;
    v[1] = g_launch[i].grid.y;
    v[2] = g_launch[i].block.x;
    v[3] = (uint32_t)g_launch[i].refused;
}
void rec_clear(void) { g_launches = 0; }

void *__hipRegisterFatBinary(const void *data) { (void)data; return g_heap; }
void __hipUnregisterFatBinary(void *m) { (void)m; }
void __hipRegisterFunction(void *m, const void *fn, char *dev, const char *name, unsigned lim, void *tid, void *bid,
                           void *bd, void *gd, int *ws) {
    (void)m; (void)dev; (void)lim; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
    if (g_kernels < kMaxKernels) {
        g_kernel[g_kernels].fn = fn;
        g_kernel[g_kernels++].name = name;
    }
}
void __hipRegisterVar(void *m, void *v, char *dev, char *name, int ext, size_t n, int c, int g) {
    (void)m; (void)v; (void)dev; (void)name; (void)ext; (void)n; (void)c; (void)g;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shared, void *stream) {
    g_config.grid = grid;
    g_config.block = block;
    g_config.shared = shared;
    g_config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shared, void **stream) {
    *grid = g_config.grid;
    *block = g_config.block;
    *shared = g_config.shared;
    *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void *fn, Dim3 grid, Dim3 block, void **args, size_t shared, void *stream) {
    (void)args; (void)shared; (void)stream;
    const char *name = "?";
    for (int i = 0; i < g_kernels; ++i)
        if (g_kernel[i].fn == fn) name = g_kernel[i].name;
    const int refused = (uint64_t)grid.x * block.x > 0xFFFFFFFFull;
    if (g_launches < kMaxLaunches) {
        g_launch[g_launches].name = name;
        g_launch[g_launches].grid = grid;
        g_launch[g_launches].block = block;
        g_launch[g_launches++].refused = refused;
    }
    if (refused) g_last = kInvalidConfiguration;
    return refused ? kInvalidConfiguration : 0;
}
int hipGetLastError(void) {
    const int e = g_last;
    g_last = 0;
    return e;
}

static int give(void **p) {
    *p = (void *)(uintptr_t)(1ull << 52);
    return 0;
}
int hipMalloc(void **p, size_t n) { (void)n; return give(p); }
int hipMallocAsync(void **p, size_t n, void *s) { (void)n; (void)s; return give(p); }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = g_heap; return n <= sizeof g_heap ? 0 : 2; }
int hipFree(void *p) { (void)p; return 0; }
int hipFreeAsync(void *p, void *s) { (void)p; (void)s; return 0; }
int hipHostFree(void *p) { (void)p; return 0; }
int hipGetSymbolAddress(void **p, const void *sym) { (void)sym; return give(p); }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipEventCreate(void **e) { *e = g_heap; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = g_heap; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventQuery(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)d; (void)s; (void)n; (void)k; (void)st; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = g_heap; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
/* graphs are not recorded: contexts that use them are outside these tests */
int hipGraphCreate(void **g, unsigned f) { (void)g; (void)f; return 801; }
int hipGraphDestroy(void *g) { (void)g; return 0; }
int hipGraphExecDestroy(void *g) { (void)g; return 0; }
int hipGraphAddKernelNode(void **n, void *g, const void *d, size_t c, const void *p) { (void)n; (void)g; (void)d; (void)c; (void)p; return 801; }
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t c) { (void)e; (void)g; (void)n; (void)l; (void)c; return 801; }
int hipGraphExecKernelNodeSetParams(void *e, void *n, const void *p) { (void)e; (void)n; (void)p; return 801; }
int hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return 801; }
