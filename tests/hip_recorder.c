/* A HIP runtime that runs nothing and records: the entry points libadiwave.so calls, so
 * that its host code (plans, dispatch, error paths) can be followed on a machine without
 * a GPU.  Loaded with global visibility before the library (tests/recorder.py).
 * "Device" memory is host memory; kernels are logged by their symbol, not run, but for
 * the reduction of the largest r, whose result rec_set_rmax gives.  Copies and fills of
 * at most 64 bytes and uploads are done, the others (between levels, which may be any
 * addresses) only logged. */
#define _GNU_SOURCE
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct { unsigned x, y, z; } dim3_t;

enum { kOk = 0, kFailed = 1, kMaxFn = 512 };
static struct { const void* fn; const char* name; } g_fn[kMaxFn];
static int g_nfn;
static char* g_log;
static size_t g_len, g_cap;
static double g_rmax;
static int g_event_countdown = -1, g_capturing;
static float g_ms[64];
static int g_nms, g_ims;

static void log_line(const char* s)
{
    const size_t n = strlen(s);
    if (g_len + n + 2 > g_cap) {
        g_cap = 2 * (g_len + n + 2);
        g_log = realloc(g_log, g_cap);
    }
    memcpy(g_log + g_len, s, n);
    g_len += n;
    g_log[g_len++] = '\n';
    g_log[g_len] = 0;
}

/* ------------------------------------------------------------ for the tests ---- */
const char* rec_log(void) { return g_log ? g_log : ""; }
void rec_clear(void)
{
    g_len = 0;
    if (g_log) g_log[0] = 0;
}
void rec_set_rmax(double r) { g_rmax = r; }
void rec_fail_event(int n) { g_event_countdown = n; }   /* the n-th record from now fails (0: the next) */
void rec_capturing(int on) { g_capturing = on; }
/* what hipEventElapsedTime gives from now on, in turn (the last one for good) */
void rec_times(const float* ms, int n)
{
    g_nms = n < 64 ? n : 64;
    g_ims = 0;
    memcpy(g_ms, ms, (size_t)g_nms * sizeof(float));
}

/* ------------------------------------------------------------- registration ---- */
void** __hipRegisterFatBinary(const void* data) { (void)data; return (void**)&g_nfn; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned lim, void* a, void* b,
                           void* c, void* d, int* e)
{
    (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (g_nfn == kMaxFn) { fprintf(stderr, "recorder: too many kernels\n"); abort(); }
    g_fn[g_nfn].fn = fn;
    g_fn[g_nfn++].name = name;
}
void __hipRegisterVar(void** m, void* v, char* hv, char* dv, int ext, size_t size, int c, int g)
{
    (void)m; (void)v; (void)hv; (void)dv; (void)ext; (void)size; (void)c; (void)g;
}

/* ----------------------------------------------------------------- launches ---- */
static struct { dim3_t grid, block; size_t shmem; void* stream; } g_cfg;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void* stream)
{
    g_cfg.grid = grid; g_cfg.block = block; g_cfg.shmem = shmem; g_cfg.stream = stream;
    return kOk;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shmem, void** stream)
{
    *grid = g_cfg.grid; *block = g_cfg.block; *shmem = g_cfg.shmem; *stream = g_cfg.stream;
    return kOk;
}
int hipLaunchKernel(const void* fn, dim3_t grid, dim3_t block, void** args, size_t shmem, void* stream)
{
    const char* name = "?";
    char line[1024];
    (void)shmem; (void)stream;
    for (int k = 0; k < g_nfn; ++k)
        if (g_fn[k].fn == fn) name = g_fn[k].name;
    if (strstr(name, "k_rmax64")) **(double**)args[2] = g_rmax;
    else if (strstr(name, "k_rmax")) **(float**)args[2] = (float)g_rmax;
    snprintf(line, sizeof line, "%s %u %u", name, grid.x * grid.y * grid.z, block.x);
    log_line(line);
    return kOk;
}

/* ------------------------------------------------------------------- memory ---- */
/* (address space only, no memory until it is touched: nothing here reads whole fields) */
int hipMalloc(void** p, size_t n)
{
    size_t* q = mmap(NULL, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED) return kFailed;
    q[0] = n + 4096;
    *p = (char*)q + 4096;
    return kOk;
}
int hipFree(void* p)
{
    if (p) munmap((char*)p - 4096, *(size_t*)((char*)p - 4096));
    return kOk;
}
int hipGetSymbolAddress(void** p, const void* sym) { (void)sym; return hipMalloc(p, (size_t)1 << 26); }
int hipMemsetAsync(void* p, int v, size_t n, void* s)
{
    (void)s;
    if (n <= 64) memset(p, v, n);
    return kOk;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st)
{
    (void)st;
    if (n <= 64 || kind == 1) memcpy(d, s, n);       /* 1: host to device */
    log_line("memcpy");
    return kOk;
}

/* ------------------------------------------- streams, events, graphs, device ---- */
static char g_handle;
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &g_handle; return kOk; }
int hipStreamDestroy(void* s) { (void)s; return kOk; }
int hipStreamSynchronize(void* s) { (void)s; return kOk; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return kOk; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = g_capturing; return kOk; }
int hipStreamBeginCapture(void* s, int m) { (void)s; (void)m; return kOk; }
int hipStreamEndCapture(void* s, void** g) { (void)s; *g = &g_handle; return kOk; }
int hipGraphInstantiate(void** e, void* g, void* n, char* b, size_t z)
{
    (void)g; (void)n; (void)b; (void)z;
    *e = &g_handle;
    return kOk;
}
int hipGraphLaunch(void* e, void* s) { (void)e; (void)s; log_line("graph"); return kOk; }
int hipGraphDestroy(void* g) { (void)g; return kOk; }
int hipGraphExecDestroy(void* e) { (void)e; return kOk; }
int hipEventCreate(void** e) { *e = &g_handle; return kOk; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = &g_handle; return kOk; }
int hipEventDestroy(void* e) { (void)e; return kOk; }
int hipEventSynchronize(void* e) { (void)e; return kOk; }
int hipEventRecord(void* e, void* s)
{
    (void)e; (void)s;
    if (g_event_countdown < 0) return kOk;
    return g_event_countdown-- == 0 ? kFailed : kOk;
}
int hipEventElapsedTime(float* ms, void* a, void* b)
{
    (void)a; (void)b;
    *ms = g_nms ? g_ms[g_ims < g_nms - 1 ? g_ims++ : g_nms - 1] : 1.0f;
    return kOk;
}
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return kOk; }
int hipGetLastError(void) { return kOk; }
const char* hipGetErrorString(int e) { return e ? "recorder: failed as asked" : "no error"; }
