/* A stand-in for the HIP runtime on a machine without a GPU: the library's host code runs
 * against it and nothing is computed.  It records kernel launches and function attributes
 * and lets device memory be host memory.  Events measure what `elapsed_of_grid` makes of
 * the last launch of a kernel whose name contains `timed_kernel`. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { MAX_FN = 4096, MAX_LOG = 65536 };
static const void* fn_ptr[MAX_FN];
static const char* fn_name[MAX_FN];
static int n_fn;

struct launch { const char* name; uint32_t grid, block; size_t shmem; };
struct launch stub_launches[MAX_LOG];
int stub_n_launches;
struct attr { const char* name; int attr, value; };
struct attr stub_attrs[MAX_LOG];
int stub_n_attrs;
const char* timed_kernel = "\n";
float (*elapsed_of_grid)(uint32_t);
static uint32_t timed_grid;

static const char* name_of(const void* f) {
    for (int i = 0; i < n_fn; ++i)
        if (fn_ptr[i] == f) return fn_name[i];
    return "?";
}

void** __hipRegisterFatBinary(const void* data) {
    static void* module;
    (void)data;
    return &module;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned n, void* a, void* b,
                           void* c, void* d, int* w) {
    (void)m, (void)dev, (void)n, (void)a, (void)b, (void)c, (void)d, (void)w;
    if (n_fn < MAX_FN) {
        fn_ptr[n_fn] = host;
        fn_name[n_fn++] = strdup(name);
    }
}
void __hipRegisterVar(void** m, void* var, char* h, char* d, int e, size_t s, int c, int g) {
    (void)m, (void)var, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
static dim3_t cfg_grid, cfg_block;
static size_t cfg_shmem;
static void* cfg_stream;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t s, void* st) {
    cfg_grid = g, cfg_block = b, cfg_shmem = s, cfg_stream = st;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* s, void** st) {
    *g = cfg_grid, *b = cfg_block, *s = cfg_shmem, *st = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t shmem, void* st) {
    (void)args, (void)st;
    const struct launch l = {name_of(f), g.x, b.x, shmem};
    if (stub_n_launches < MAX_LOG) stub_launches[stub_n_launches++] = l;
    if (strstr(l.name, timed_kernel)) timed_grid = g.x;
    return 0;
}
int hipFuncSetAttribute(const void* f, int attr, int value) {
    const struct attr a = {name_of(f), attr, value};
    if (stub_n_attrs < MAX_LOG) stub_attrs[stub_n_attrs++] = a;
    return 0;
}
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) {
    (void)e;
    return "stub";
}
int hipGetDevice(int* d) { return *d = 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) {
    (void)attr, (void)dev;
    *v = 256;
    return 0;
}
int hipMalloc(void** p, size_t n) {
    *p = calloc(n ? n : 1, 1);
    return 0;
}
int hipFree(void* p) {
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned f) {
    (void)f;
    return hipMalloc(p, n);
}
int hipHostFree(void* p) { return hipFree(p); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
    (void)kind, (void)st;
    memcpy(d, s, n);
    return 0;
}
int hipStreamSynchronize(void* st) {
    (void)st;
    return 0;
}
int hipEventCreate(void** e) { return hipMalloc(e, 1); }
int hipEventDestroy(void* e) { return hipFree(e); }
int hipEventRecord(void* e, void* st) {
    (void)e, (void)st;
    return 0;
}
int hipEventSynchronize(void* e) {
    (void)e;
    return 0;
}
int hipEventElapsedTime(float* ms, void* a, void* b) {
    (void)a, (void)b;
    *ms = elapsed_of_grid ? elapsed_of_grid(timed_grid) : 1.0f;
    return 0;
}
