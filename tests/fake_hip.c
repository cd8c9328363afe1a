/* A stand-in for the HIP runtime, for host-side tests without a GPU: device
 * memory is host memory, kernels do not run, every timed span takes 1 ms.
 * fake_hip_fail_above(n): device allocations above n bytes fail (0: none).
 * fake_hip_log(): one line per kernel launch, "name grid block units" (units:
 * the persistent kernel's number of work units, else 0). */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

static size_t fail_above;
static int last_error, n_fun;
static struct { const void* f; const char* name; } fun[4096];
static char log_buf[1 << 20];
static size_t log_n;
static struct { dim3_t g, b; size_t shm; void* st; } cfg;

void fake_hip_fail_above(size_t n) { fail_above = n; }
const char* fake_hip_log(void) { return log_buf; }
void fake_hip_clear(void) { log_n = 0; log_buf[0] = 0; }

static int alloc(void** p, size_t n)
{
    *p = NULL;
    if (fail_above && n > fail_above) return last_error = 2; /* hipErrorOutOfMemory */
    *p = calloc(n ? n : 1, 1);
    return *p ? 0 : (last_error = 2);
}
int hipMalloc(void** p, size_t n) { return alloc(p, n); }
int hipMallocAsync(void** p, size_t n, void* st) { (void)st; return alloc(p, n); }
int hipHostMalloc(void** p, size_t n, unsigned fl) { (void)fl; *p = calloc(n, 1); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipFreeAsync(void* p, void* st) { (void)st; free(p); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipEventCreate(void** e) { *e = &cfg; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = &cfg; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* st) { (void)e; (void)st; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.0f; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &cfg; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t s)
{
    (void)f; (void)s;
    *n = 1024 / b; /* four waves per SIMD */
    return 0;
}
void** __hipRegisterFatBinary(const void* d) { (void)d; return (void**)&cfg; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* n, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* f, char* h, const char* name, unsigned t, void* a, void* b, void* c,
                           void* d, int* w)
{
    (void)m; (void)h; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (n_fun < 4096) { fun[n_fun].f = f; fun[n_fun++].name = strdup(name); }
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t shm, void* st)
{
    cfg.g = g; cfg.b = b; cfg.shm = shm; cfg.st = st;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* shm, void** st)
{
    *g = cfg.g; *b = cfg.b; *shm = cfg.shm; *st = cfg.st;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t shm, void* st)
{
    const char* name = "?";
    long long units = 0;
    (void)shm; (void)st;
    for (int i = 0; i < n_fun; ++i)
        if (fun[i].f == f) name = fun[i].name;
    if (strstr(name, "persistent_kernel")) units = *(const int64_t*)args[5];
    if (log_n < sizeof(log_buf) - 1024)
        log_n += (size_t)snprintf(log_buf + log_n, 1024, "%.900s %u %u %lld\n", name, g.x, b.x, units);
    return 0;
}
