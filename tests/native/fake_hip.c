// A stand-in for the HIP runtime calls of libmnufft, for tests of its host code on
// machines without a GPU: device memory is address space that nothing touches,
// kernels do not run, and what the library asks for is recorded.  Loaded with
// RTLD_GLOBAL before the library (tests/host_shim.py).
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
enum { kOk = 0, kOutOfMemory = 2 };

// ---- device memory ----------------------------------------------------------
enum { kBlocks = 1 << 16 };
static struct { uintptr_t base; size_t bytes; int live, dev; } blk[kBlocks];
static int nblk, device;
static uintptr_t next_base = (uintptr_t)1 << 44;
static long long live_bytes, capacity = -1;
static long counts[16];
enum { C_MALLOC, C_FREE, C_STREAM_SYNC, C_DEVICE_SYNC, C_LAUNCH, C_OVERRUN, C_SYNC_DEV, C_QUEUE };

long fake_count(int what) { return counts[what]; }
void fake_clear(void) { memset(counts, 0, sizeof(counts)); }
long long fake_live(void) { return live_bytes; }
void fake_capacity(long long bytes) { capacity = bytes; }  // of all live blocks; < 0: none

static size_t room(uintptr_t p)  // bytes from p to the end of its live block
{
    for (int i = nblk - 1; i >= 0; --i)
        if (blk[i].live && p >= blk[i].base && p < blk[i].base + blk[i].bytes)
            return blk[i].base + blk[i].bytes - p;
    return 0;
}
static void need(const char *what, const void *p, size_t bytes)
{
    if (bytes && p && room((uintptr_t)p) < bytes) {
        ++counts[C_OVERRUN];
        fprintf(stderr, "overrun: %s: %zu bytes in %zu\n", what, bytes, room((uintptr_t)p));
    }
}

int hipMalloc(void **p, size_t n)
{
    ++counts[C_MALLOC];
    if (nblk == kBlocks || (capacity >= 0 && live_bytes + (long long)n > capacity)) return kOutOfMemory;
    blk[nblk].base = next_base;
    blk[nblk].bytes = n;
    blk[nblk].live = 1;
    blk[nblk].dev = device;
    ++nblk;
    *p = (void *)next_base;
    next_base += (n + 4095) / 4096 * 4096 + 4096;
    live_bytes += (long long)n;
    return kOk;
}
int hipFree(void *p)
{
    ++counts[C_FREE];
    for (int i = nblk - 1; i >= 0; --i)
        if (blk[i].live && blk[i].base == (uintptr_t)p) {
            blk[i].live = 0;
            live_bytes -= (long long)blk[i].bytes;
            return kOk;
        }
    return 1;
}
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return kOk; }
int hipHostFree(void *p) { free(p); return kOk; }
// device to host gives zeros; type 3 bounds (18 doubles: least, largest and a flag
// per dimension and set) the ones set here
static double bounds;
void fake_bounds(double b) { bounds = b; }
int hipMemcpy(void *d, const void *s, size_t n, int kind)
{
    (void)s;
    if (kind != 2) return kOk;
    memset(d, 0, n);
    for (int k = 0; n == 18 * 8 && k < 6; ++k) {
        ((double *)d)[3 * k] = -bounds;
        ((double *)d)[3 * k + 1] = bounds;
    }
    return kOk;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { (void)st; return hipMemcpy(d, s, n, kind); }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; return hipMalloc(p, 1 << 20); }

// std::chrono::steady_clock::now: the time that the test sets
static long long clock_ns;
void fake_time(double seconds) { clock_ns = (long long)(seconds * 1e9); }
long long _ZNSt6chrono3_V212steady_clock3nowEv(void) { return clock_ns; }

// ---- devices, streams, events --------------------------------------------------
static void *capturing;
void fake_capture(void *stream) { capturing = stream; }
int hipGetDevice(int *d) { *d = device; return kOk; }
int hipSetDevice(int d) { device = d; return kOk; }
int hipGetLastError(void) { return kOk; }
static int failing;
void fake_fail_waits(int on) { failing = on; }
int hipDeviceSynchronize(void) { ++counts[C_DEVICE_SYNC]; counts[C_SYNC_DEV] = device; return failing; }
int hipStreamSynchronize(void *s) { (void)s; ++counts[C_STREAM_SYNC]; counts[C_SYNC_DEV] = device; return failing; }
static void *gone;
void fake_stream_gone(void *stream) { gone = stream; }  // using it counts as an overrun
int hipStreamIsCapturing(void *s, int *st)
{
    if (s && s == gone) ++counts[C_OVERRUN];
    *st = s && s == capturing;
    return kOk;
}
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return kOk; }
int hipStreamDestroy(void *s) { free(s); return kOk; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return kOk; }
int hipEventCreate(void **e) { *e = malloc(1); return kOk; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return kOk; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return kOk; }
int hipEventSynchronize(void *e) { (void)e; return kOk; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1; return kOk; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return kOk; }

// ---- kernels --------------------------------------------------------------------
static struct { const void *fn; const char *name; } fns[8192];
static int nfn;
static int dummy;
void **__hipRegisterFatBinary(const void *d) { (void)d; return (void **)&dummy; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void *m, void *v, char *h, char *n, int e, size_t z, int c, int g)
{
    (void)m; (void)v; (void)h; (void)n; (void)e; (void)z; (void)c; (void)g;
}
void __hipRegisterFunction(void *m, const void *fn, char *h, const char *name, unsigned l, void *t,
                           void *b, void *bd, void *gd, int *w)
{
    (void)m; (void)h; (void)l; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (nfn < 8192) {
        fns[nfn].fn = fn;
        fns[nfn++].name = strdup(name);
    }
}
static dim3_t cg, cb;
static size_t csh;
static void *cst;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void *st)
{
    cg = g; cb = b; csh = sh; cst = st;
    return kOk;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *sh, void **st)
{
    *g = cg; *b = cb; *sh = csh; *st = cst;
    return kOk;
}

// What a kernel writes, by its arguments, against the block that it writes to.
#define I32(k) (*(int *)args[k])
#define PTR(k) (*(void **)args[k])
int hipLaunchKernel(const void *fn, dim3_t g, dim3_t b, void **args, size_t sh, void *st)
{
    (void)b; (void)sh; (void)st;
    ++counts[C_LAUNCH];
    const char *n = "";
    for (int i = 0; i < nfn; ++i)
        if (fns[i].fn == fn) n = fns[i].name;
    if (strstr(n, "k_radix_hist")) {        // (keys or points, M, shift, dmask, pitch, hist)
        need(n, PTR(5), (size_t)256 * I32(4) * 4);
        if (I32(4) < (int)g.x) need("columns of k_radix_hist", PTR(5), ~(size_t)0 / 2);
    }
    if (strstr(n, "k_scan_reduce")) need(n, PTR(2), (size_t)g.x * 4);  // (in, n, partials)
    if (strstr(n, "k_scan_down")) need(n, PTR(1), *(size_t *)args[2] * 4);  // (in, out, n, partials)
    // (geometry, sub, nsub, u0, u1, u2, index, grid, c, bk, work, ..)
    if (strstr(n, "k_interp_mf") && PTR(10)) ++counts[C_QUEUE];
    // 160 KB of LDS, some of it static
    if (strstr(n, "_mf") && sh + 16 > 160 * 1024) need("LDS of a matrix-core kernel", (void *)1, 1);
    if (strstr(n, "k_subfill")) {           // (nbins, msub, nsub_max, .., .., sub, .., mergelist)
        need(n, PTR(5), (size_t)I32(2) * 16);
        need(n, PTR(10), (size_t)I32(2) * 4);
    }
    return kOk;
}
