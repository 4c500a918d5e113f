/* A HIP runtime that does nothing, for host tests of libsnrt's launch
 * sequences: loaded (RTLD_GLOBAL) before the library, its functions stand in
 * for libamdhip64's. It keeps the list of launches (kernel, grid, block, LDS) and
 * can make the k-th call of a function fail. No device memory is touched, so
 * any address will do for a buffer. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
enum { OK = 0, OUT_OF_MEMORY = 2, MAX_LAUNCHES = 4096 };

static struct { const void* kernel; unsigned long long blocks, threads, shared; } launches[MAX_LAUNCHES];
static int n_launches, graph_replays;
static char fail_name[64];
static int fail_at;
static dim3_t grid_, block_;
static size_t shared_;
static void* stream_;

static int status(const char* name) {
    if (fail_at > 0 && strcmp(name, fail_name) == 0 && --fail_at == 0) return OUT_OF_MEMORY;
    return OK;
}
#define CALL return status(__func__)

/* for the test */
void stub_clear(void) { n_launches = graph_replays = 0; }
void stub_fail(const char* name, int k) {
    snprintf(fail_name, sizeof fail_name, "%s", name);
    fail_at = k;
}
int stub_launches(void) { return n_launches; }
int stub_graph_replays(void) { return graph_replays; }
const char* stub_kernel(int i) {
    Dl_info d;
    return dladdr(launches[i].kernel, &d) && d.dli_sname ? d.dli_sname : "?";
}
unsigned long long stub_blocks(int i) { return launches[i].blocks; }
unsigned long long stub_threads(int i) { return launches[i].threads; }
unsigned long long stub_shared(int i) { return launches[i].shared; }

/* launches */
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void* s) {
    grid_ = g, block_ = b, shared_ = sh, stream_ = s;
    return OK;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* sh, void** s) {
    *g = grid_, *b = block_, *sh = shared_, *s = stream_;
    return OK;
}
static int last;
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t sh, void* s) {
    (void)args, (void)s;
    if (n_launches < MAX_LAUNCHES) {
        launches[n_launches].kernel = f;
        launches[n_launches].blocks = (unsigned long long)g.x * g.y * g.z;
        launches[n_launches].threads = (unsigned long long)b.x * b.y * b.z;
        launches[n_launches].shared = sh;
        n_launches++;
    }
    return last = status(__func__);
}
int hipGetLastError(void) {
    const int e = last;
    last = OK;
    return e;
}
int hipGraphLaunch(void* e, void* s) {
    (void)e, (void)s;
    const int st = status(__func__);
    graph_replays += st == OK;
    return st;
}

/* the rest */
static char handle[64];
const char* hipGetErrorString(int e) { return e == OK ? "ok" : "made to fail"; }
int hipGetDevice(int* d) { *d = 0; CALL; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a, (void)d; *v = 256; CALL; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t sh) {
    (void)f, (void)b, (void)sh;
    *n = 2;
    CALL;
}
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)0x700000000000; CALL; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)d, (void)s, (void)n, (void)k; CALL; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* q) { (void)d, (void)s, (void)n, (void)k, (void)q; CALL; }
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k, void* q) {
    (void)d, (void)dp, (void)s, (void)sp, (void)w, (void)h, (void)k, (void)q;
    CALL;
}
int hipMemsetAsync(void* d, int v, size_t n, void* q) { (void)d, (void)v, (void)n, (void)q; CALL; }
static char pinned[1 << 24];
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = pinned; return n <= sizeof pinned ? status(__func__) : OUT_OF_MEMORY; }
int hipHostFree(void* p) { (void)p; CALL; }
int hipEventCreate(void** e) { *e = handle; CALL; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = handle; CALL; }
int hipEventDestroy(void* e) { (void)e; CALL; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a, (void)b; *ms = 0; CALL; }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; CALL; }
int hipEventSynchronize(void* e) { (void)e; CALL; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = handle; CALL; }
int hipStreamDestroy(void* s) { (void)s; CALL; }
int hipStreamSynchronize(void* s) { (void)s; CALL; }
int hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; CALL; }
int hipStreamEndCapture(void* s, void** g) { (void)s; *g = handle; CALL; }
int hipGraphInstantiate(void** e, void* g, void* n, char* l, size_t z) { (void)g, (void)n, (void)l, (void)z; *e = handle; CALL; }
int hipGraphExecDestroy(void* e) { (void)e; CALL; }
int hipGraphDestroy(void* g) { (void)g; CALL; }
