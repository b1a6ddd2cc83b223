/* A HIP runtime that runs nothing and records every kernel launch, preloaded by
 * test_launches.py: what a call launches (kernel, grid, threads, LDS, stream) is
 * decided on the host and can be read on a machine without a GPU.  Copies to
 * and from the device are skipped, every call succeeds. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_;
typedef void *ptr;

struct record { char name[512]; uint32_t grid[3], block[3]; uint64_t lds; uint64_t stream; };
static struct record recs[4096];
static int nrecs;
static uintptr_t next_handle = 0x1000;
static int last_error;

int rec_count(void) { return nrecs; }
void rec_clear(void) { nrecs = 0; }
const struct record *rec_get(int i) { return &recs[i]; }

int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t lds, ptr stream)
{
    (void)args;
    Dl_info info;
    if (nrecs < 4096) {
        struct record *r = &recs[nrecs++];
        const char *name = dladdr(f, &info) && info.dli_sname ? info.dli_sname : "?";
        snprintf(r->name, sizeof r->name, "%s", name);
        r->grid[0] = g.x; r->grid[1] = g.y; r->grid[2] = g.z;
        r->block[0] = b.x; r->block[1] = b.y; r->block[2] = b.z;
        r->lds = lds;
        r->stream = (uint64_t)(uintptr_t)stream;
    }
    /* the runtime's own limit: fewer than 2^32 threads in a dimension of the grid */
    if ((uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32 || (uint64_t)g.z * b.z >> 32) return last_error = 9;
    return 0;
}

static _Thread_local struct { dim3_ g, b; size_t lds; ptr stream; } conf;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t lds, ptr stream)
{
    conf.g = g; conf.b = b; conf.lds = lds; conf.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *lds, ptr *stream)
{
    *g = conf.g; *b = conf.b; *lds = conf.lds; *stream = conf.stream;
    return 0;
}

static int handle(ptr *out) { *out = (ptr)(next_handle += 0x100); return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipEventCreate(ptr *e) { return handle(e); }
int hipEventCreateWithFlags(ptr *e, unsigned f) { (void)f; return handle(e); }
int hipEventDestroy(ptr e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, ptr a, ptr b) { (void)a; (void)b; *ms = 1; return 0; }
int hipEventQuery(ptr e) { (void)e; return 0; }
int hipEventRecord(ptr e, ptr s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(ptr e) { (void)e; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetDevicePropertiesR0600(char *p, int d) { (void)d; memset(p, 0, 1472); strcpy(p, "recorder"); return 0; }
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipGetSymbolAddress(ptr *p, const void *s) { (void)s; *p = (ptr)((uintptr_t)1 << 44); return 0; }
int hipHostMalloc(ptr *p, size_t n, unsigned f) { (void)n; (void)f; *p = NULL; return 2; }
int hipLaunchHostFunc(ptr s, void (*fn)(void *), void *arg) { (void)s; fn(arg); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)d; (void)s; (void)n; (void)k; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, ptr st) { (void)d; (void)s; (void)n; (void)k; (void)st; return 0; }
int hipMemsetAsync(void *d, int v, size_t n, ptr st) { (void)d; (void)v; (void)n; (void)st; return 0; }
int hipStreamCreateWithFlags(ptr *s, unsigned f) { (void)f; return handle(s); }
int hipStreamDestroy(ptr s) { (void)s; return 0; }
int hipStreamSynchronize(ptr s) { (void)s; return 0; }
int hipStreamWaitEvent(ptr s, ptr e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipStreamIsCapturing(ptr s, int *st) { (void)s; *st = 0; return 0; }
int hipStreamGetCaptureInfo_v2(ptr s, int *st, unsigned long long *id, ptr *g, const ptr **deps, size_t *nd)
{
    (void)s;
    if (st) *st = 0;
    if (id) *id = 0;
    if (g) *g = NULL;
    if (deps) *deps = NULL;
    if (nd) *nd = 0;
    return 0;
}
