/* The HIP calls of libkdcd.so's host code on host memory: kernels are logged by name and
 * not run (but for the fill kernel), streams and captures are flags that a test sets.
 * Loaded before the library with global symbols, it takes the runtime's place. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { const void *f; const char *name; } Fn;
typedef struct { void *p; size_t n; int captured; } Block;

static Fn fns[4096];
static int n_fns;
static Block blocks[4096];
static int n_blocks;
static struct { dim3 g, b; size_t sh; void *st; } cfg;
static char launched[1 << 20];

/* set by the test */
int stub_capturing, stub_sync_error, stub_coop_refused, stub_coop_gives_up;
uint64_t stub_row_max;                       /* the longest CSR row */
size_t stub_memory = (size_t)1 << 40;
/* read by the test */
int stub_mallocs, stub_captured_mallocs, stub_uses_captured, stub_coop_launches;
size_t stub_held, stub_largest;

const char *stub_launched(void) { return launched; }
void stub_forget(void) { launched[0] = 0; stub_mallocs = 0; stub_coop_launches = 0; stub_largest = 0; }

static const char *name_of(const void *f)
{
    for (int i = 0; i < n_fns; ++i)
        if (fns[i].f == f) return fns[i].name;
    return "?";
}
static int inside(const Block *b, const void *p)
{
    return (const char *)p >= (const char *)b->p && (const char *)p < (const char *)b->p + b->n;
}
/* an address of memory that only a captured graph may touch (reads 8 bytes an argument:
 * arguments lie in the caller's frames) */
static void look_at(void **args, int n)
{
    for (int a = 0; a < n; ++a)
        for (int i = 0; i < n_blocks; ++i)
            if (!stub_capturing && blocks[i].p && blocks[i].captured && inside(&blocks[i], *(void **)args[a])) ++stub_uses_captured;
}

static int launch(const void *f, void **args)
{
    const char *name = name_of(f);
    if (strlen(launched) + strlen(name) + 2 < sizeof launched) {
        strcat(launched, name);
        strcat(launched, " ");
    }
    if (strstr(name, "fill_i32")) {
        look_at(args, 1);
        if (!stub_capturing) {
            int32_t *p = *(int32_t **)args[0];
            const int32_t v = *(int32_t *)args[1];
            const int64_t c = *(int64_t *)args[2];
            for (int64_t i = 0; i < c; ++i) p[i] = v;
        }
    }
    if (strstr(name, "csr_row_max") && !stub_capturing) **(uint64_t **)args[2] = stub_row_max;
    return 0;
}

void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, ...) { (void)h; }
void __hipRegisterFunction(void **h, const void *f, char *df, const char *dn, unsigned t, void *a, void *b, void *c, void *d, int *w)
{
    (void)h; (void)df; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (n_fns < 4096) fns[n_fns++] = (Fn){f, dn};
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, void *st) { cfg.g = g; cfg.b = b; cfg.sh = sh; cfg.st = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, void **st) { *g = cfg.g; *b = cfg.b; *sh = cfg.sh; *st = cfg.st; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t sh, void *st) { (void)g; (void)b; (void)sh; (void)st; return launch(f, args); }
int hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t sh, void *st, void *e0, void *e1, int fl)
{
    (void)g; (void)b; (void)sh; (void)st; (void)e0; (void)e1; (void)fl;
    return launch(f, args);
}
/* the cooperative kernel's arguments end with alpha, trace, slots, status (and what the
 * library adds after them): a launch that gives up has spoilt alpha */
int hipLaunchCooperativeKernel(const void *f, dim3 g, dim3 b, void **args, unsigned sh, void *st)
{
    (void)g; (void)b; (void)sh; (void)st;
    if (stub_coop_refused) return 720;
    ++stub_coop_launches;
    launch(f, args);
    if (stub_coop_gives_up) {
        (*(double **)args[12])[0] = -77.0;
        **(int32_t **)args[15] = -1000;
    }
    return 0;
}

static int alloc(void **p, size_t n, int captured)
{
    *p = 0;
    if (stub_held + n > stub_memory || n_blocks == 4096) return 2;
    if (posix_memalign(p, 4096, n ? n : 1)) return 2;
    memset(*p, 0, n);
    blocks[n_blocks++] = (Block){*p, n, captured};
    stub_held += n;
    if (captured) ++stub_captured_mallocs; else ++stub_mallocs;
    if (n > stub_largest) stub_largest = n;
    return 0;
}
int hipFree(void *p)
{
    for (int i = 0; i < n_blocks; ++i)
        if (p && blocks[i].p == p) {
            stub_held -= blocks[i].n;
            if (!blocks[i].captured) { free(p); blocks[i].p = 0; }
        }
    return 0;
}
int hipMalloc(void **p, size_t n) { return alloc(p, n, 0); }
int hipMallocAsync(void **p, size_t n, void *st) { (void)st; return alloc(p, n, stub_capturing); }
int hipFreeAsync(void *p, void *st) { (void)st; return hipFree(p); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st)
{
    (void)kind; (void)st;
    if (!stub_capturing) memcpy(d, s, n);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) { return hipMemcpyAsync(d, s, n, kind, 0); }
int hipStreamSynchronize(void *st) { (void)st; return stub_capturing ? 900 : stub_sync_error; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamIsCapturing(void *st, int *s) { (void)st; *s = stub_capturing ? 1 : 0; return 0; }
int hipStreamGetDevice(void *st, int *d) { (void)st; *d = 0; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int t, size_t s) { (void)f; (void)t; (void)s; *n = 1; return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *st) { (void)e; (void)st; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 1.f; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
/* graphs: a private stream's capture, whose memory is the caller's */
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return 0; }
int hipStreamBeginCapture(void *s, int m) { (void)s; (void)m; return 0; }
int hipStreamEndCapture(void *s, void **g) { (void)s; *g = malloc(1); return 0; }
int hipGraphInstantiate(void **x, void *g, void **n, char *l, size_t z) { (void)g; (void)n; (void)l; (void)z; *x = malloc(1); return 0; }
int hipGraphDestroy(void *g) { free(g); return 0; }
int hipGraphExecDestroy(void *x) { free(x); return 0; }
int hipGraphLaunch(void *x, void *s) { (void)x; (void)s; return 0; }
