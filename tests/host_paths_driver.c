/* Host side of libpulbm.so against a stand-in HIP runtime: device memory is host
 * memory, kernels do nothing (k_pack_rows copies its rows), and the runtime's
 * rules that matter here are kept: an event is recorded on streams of its own
 * device only, allocations and frees are refused during another stream's
 * capture unless the thread is in relaxed mode, pinned memory can run out.
 * The executable's symbols come before libamdhip64's in the library's lookup.
 *
 *   host_paths <libpulbm.so> <scenario> [arguments]
 */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "pulbm.h"

typedef struct { uint32_t x, y, z; } dim3;
typedef struct { int device; } Stream;
typedef struct { int device; unsigned flags; } Event;
enum { kInvalid = 1, kNoMemory = 2, kInvalidHandle = 400, kCaptureUnsupported = 900 };
enum { kPortable = 1, kCoherent = 0x40000000 };
static const unsigned kReleaseToSystem = 0x80000000u;

static __thread int device, mode, last_error;
static int capturing, pinned_left = 1 << 30, pinned_live, pinned_incoherent, events_loose, refused, launches;
static struct { const void* f; char name[200]; } kernels[400];
static int nkernels;
static char watch[64];
static size_t watched_lds[64];
static int nwatched;

static int ret(int e)
{
    if (e) last_error = e;
    return e;
}
static int allowed(void)
{
    if (!capturing || mode == 2) return 1;
    __sync_fetch_and_add(&refused, 1);
    return 0;
}

void** __hipRegisterFatBinary(const void* d) { (void)d; return calloc(1, 8); }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g)
{
    (void)m, (void)v, (void)h, (void)d, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void** m, const void* f, char* dn, const char* name, unsigned t, void* a, void* b, void* c,
                           void* d, int* w)
{
    (void)m, (void)dn, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
    kernels[nkernels].f = f;
    strncpy(kernels[nkernels++].name, name, 199);
}
static __thread struct { dim3 g, b; size_t lds; void* st; } call;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* st)
{
    call.g = g, call.b = b, call.lds = lds, call.st = st;
    return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** st)
{
    *g = call.g, *b = call.b, *lds = call.lds, *st = call.st;
    return 0;
}

typedef struct { const void* f[5]; } Src;
static void pack_rows(void** a, int width)
{
    const Src* s = a[0];
    int f0 = *(int*)a[1];
    uint32_t row0 = *(uint32_t*)a[2], i0 = *(uint32_t*)a[3], rows = *(uint32_t*)a[4], nx = *(uint32_t*)a[5];
    uint32_t sx = *(uint32_t*)a[6], count = *(uint32_t*)a[7];
    char* out = *(char**)a[8];
    for (uint32_t k = 0; k < count; ++k) {
        uint32_t e = i0 + k, r = row0 + e / nx;
        int f = f0;
        for (; r >= rows; r -= rows) ++f;
        memcpy(out + (size_t)k * width, (const char*)s->f[f] + ((size_t)r * sx + e % nx) * width, width);
    }
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* st)
{
    (void)g, (void)b, (void)st;
    __sync_fetch_and_add(&launches, 1);
    for (int k = 0; k < nkernels; ++k)
        if (kernels[k].f == f) {
            if (strstr(kernels[k].name, "k_pack_rows")) pack_rows(args, strstr(kernels[k].name, "k_pack_rowsId") ? 8 : 4);
            if (watch[0] && strstr(kernels[k].name, watch) && nwatched < 64) watched_lds[nwatched++] = lds;
        }
    return 0;
}

int hipMalloc(void** p, size_t n)
{
    if (!allowed()) return ret(kCaptureUnsupported);
    return posix_memalign(p, 256, n ? n : 1) ? ret(kNoMemory) : 0;
}
int hipFree(void* p)
{
    if (!allowed()) return ret(kCaptureUnsupported);
    free(p);
    return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned flags)
{
    if (!allowed()) return ret(kCaptureUnsupported);
    if (__sync_fetch_and_sub(&pinned_left, 1) <= 0) return ret(kNoMemory);
    if (!(flags & kCoherent)) __sync_fetch_and_add(&pinned_incoherent, 1);
    __sync_fetch_and_add(&pinned_live, 1);
    *p = malloc(n);
    return 0;
}
int hipHostFree(void* p)
{
    if (!allowed()) return ret(kCaptureUnsupported);
    __sync_fetch_and_sub(&pinned_live, 1);
    __sync_fetch_and_add(&pinned_left, 1);
    free(p);
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st)
{
    (void)kind, (void)st;
    memcpy(d, s, n);
    return 0;
}
int hipGetSymbolAddress(void** p, const void* s) { (void)p, (void)s; return ret(kInvalid); }
int hipGetDevice(int* d) { *d = device; return 0; }
int hipSetDevice(int d) { device = d; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f)
{
    (void)f;
    Stream* n = malloc(sizeof *n);
    n->device = device;
    *s = n;
    return 0;
}
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; return ret(kInvalid); }
int hipStreamEndCapture(void* s, void** g) { (void)s, (void)g; return ret(kInvalid); }
int hipGraphInstantiate(void** e, void* g, void* n, char* b, size_t l) { (void)e, (void)g, (void)n, (void)b, (void)l; return ret(kInvalid); }
int hipGraphLaunch(void* e, void* s) { (void)e, (void)s; return ret(kInvalid); }
int hipGraphDestroy(void* g) { (void)g; return 0; }
int hipGraphExecDestroy(void* g) { (void)g; return 0; }
int hipThreadExchangeStreamCaptureMode(int* m)
{
    int was = mode;
    mode = *m;
    *m = was;
    return 0;
}
int hipEventCreateWithFlags(void** e, unsigned flags)
{
    Event* n = malloc(sizeof *n);
    n->device = device;
    n->flags = flags;
    *e = n;
    return 0;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s)
{
    if (((Event*)e)->device != (s ? ((Stream*)s)->device : device)) return ret(kInvalidHandle);
    return 0;
}
int hipEventSynchronize(void* e)
{
    if (!(((Event*)e)->flags & kReleaseToSystem)) __sync_fetch_and_add(&events_loose, 1);
    return 0;
}
int hipEventQuery(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* t, void* a, void* b) { (void)a, (void)b; *t = 0; return 0; }
int hipGetLastError(void)
{
    int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int e)
{
    static __thread char s[32];
    snprintf(s, sizeof s, "error %d", e);
    return s;
}

/* ------------------------------------------------------------ scenarios */

#define USE(r, name, ...) r (*name)(__VA_ARGS__)
static USE(int, required, const pulbm_params*, size_t*);
static USE(int, create, const pulbm_params*, void*, size_t, void*, pulbm_case**);
static USE(int, init, pulbm_case*, const double*, const double*, const double*);
static USE(int, step, pulbm_case*, int64_t);
static USE(int, rd, pulbm_case*, double*, double*, double*);
static USE(void, destroy, pulbm_case*);
static USE(const char*, err, void);

static pulbm_params params(int dim, int nx, int ny, int nz, int store)
{
    pulbm_params p;
    memset(&p, 0, sizeof p);
    p.dim = dim, p.nx = nx, p.ny = ny, p.nz = nz, p.store = store;
    p.q_hydro = dim == 2 ? 9 : 27, p.q_phase = dim == 2 ? 9 : 19;
    p.delta_theta = 1, p.rho_heavy = 10, p.rho_light = 1, p.nu_heavy = p.nu_light = 0.1, p.sigma = 0.01, p.W = 4;
    p.M = 0.166, p.lambda_bulk = 1. / 6;
    return p;
}

static void fail(const char* what)
{
    printf("FAILED: %s (%s)\n", what, err ? err() : "");
    exit(1);
}

/* A case in an arena of its own, every field of it filled with numbers. */
typedef struct { pulbm_case* c; char* arena; size_t n, dim; Stream st; } Made;
static void make(Made* m, const pulbm_params* p)
{
    size_t bytes = 0;
    m->n = (size_t)p->nx * p->ny * p->nz, m->dim = p->dim;
    m->st.device = device;
    if (required(p, &bytes)) fail("required_bytes");
    if (posix_memalign((void**)&m->arena, 256, bytes)) fail("arena");
    if (create(p, m->arena, bytes, &m->st, &m->c)) fail("create");
    double* z = calloc((2 + m->dim) * m->n, sizeof *z);
    if (init(m->c, z, z + m->n, z + 2 * m->n)) fail("init");
    free(z);
    if (p->store == PULBM_STORE_FP64)
        for (size_t i = 0; i < bytes / 8; ++i) ((double*)m->arena)[i] = (double)(i * 2654435761u % 1000003) * 1e-3;
    else
        for (size_t i = 0; i < bytes / 4; ++i) ((float*)m->arena)[i] = (float)(i * 2654435761u % 1000003) * 1e-3f;
}
static double* get(Made* m)
{
    double* o = malloc((2 + m->dim) * m->n * sizeof *o);
    memset(o, 0xff, (2 + m->dim) * m->n * sizeof *o);
    if (rd(m->c, o, o + m->n, o + 2 * m->n)) fail("read_fields");
    return o;
}
static void drop(Made* m)
{
    destroy(m->c);
    free(m->arena);
}
static void same(const Made* m, double* a, double* b)
{
    if (memcmp(a, b, (2 + m->dim) * m->n * sizeof *a)) fail("other values");
    free(b);
}

int main(int argc, char** argv)
{
    if (argc < 3) return 2;
    void* h = dlopen(argv[1], RTLD_NOW);
    if (!h) {
        printf("%s\n", dlerror());
        return 2;
    }
    required = dlsym(h, "pulbm_required_bytes");
    create = dlsym(h, "pulbm_create");
    init = dlsym(h, "pulbm_init_fields");
    step = dlsym(h, "pulbm_step");
    rd = dlsym(h, "pulbm_read_fields");
    destroy = dlsym(h, "pulbm_destroy");
    err = dlsym(h, "pulbm_last_error");
    const char* s = argv[2];
    /* one piece, several pieces on one thread, several threads; padded rows */
    const pulbm_params sizes[3] = {params(2, 37, 29, 1, PULBM_STORE_FP64), params(3, 61, 47, 33, PULBM_STORE_FP32),
                                   params(3, 131, 83, 51, PULBM_STORE_FP16)};
    if (!strcmp(s, "lds")) {  /* <kernel> <dim> <nx> <ny> <nz> <store> <wall> <block> <steps> [<collision>] */
        pulbm_params p = params(atoi(argv[4]), atoi(argv[5]), atoi(argv[6]), atoi(argv[7]), atoi(argv[8]));
        for (int a = 0; a < p.dim; ++a) p.wall[a] = atoi(argv[9]);
        if (atoi(argv[10]))
            for (int a = 0; a < 3; ++a) p.block_lo[a] = a < p.dim ? 2 : 0, p.block_hi[a] = a < p.dim ? 5 : 1;
        p.collision = argc > 12 ? atoi(argv[12]) : 0;
        size_t bytes = 0;
        pulbm_case* c = NULL;
        if (required(&p, &bytes)) fail("required_bytes");
        double* z = calloc((size_t)5 * p.nx * p.ny * p.nz, sizeof *z);
        const size_t n = (size_t)p.nx * p.ny * p.nz;
        if (create(&p, NULL, 0, NULL, &c) || init(c, z, z + n, z + 2 * n)) fail("case");
        strncpy(watch, argv[3], 63);
        if (step(c, atoi(argv[11]))) fail("step");
        for (int k = 0; k < nwatched; ++k) printf("%zu\n", watched_lds[k]);
        return 0;
    }
    for (int k = 0; k < 3; ++k) {
        Made m;
        make(&m, &sizes[k]);
        double* want = get(&m);
        same(&m, want, get(&m));
        if (!strcmp(s, "coherent")) {
            if (pinned_incoherent && events_loose) fail("the host may see stale pinned memory");
        } else if (!strcmp(s, "device")) {
            device = 1;
            same(&m, want, get(&m));
            if (device != 1) fail("current device changed");
            device = 0;
        } else if (!strcmp(s, "nopinned") || !strcmp(s, "onepinned")) {
            destroy(m.c);  /* gives the pieces back */
            free(m.arena);
            if (pinned_live) fail("pinned memory left");
            pinned_left = s[0] == 'o';
            make(&m, &sizes[k]);
            same(&m, want, get(&m));
            same(&m, want, get(&m));
            if (hipGetLastError()) fail("an error is left for the next call");
            pinned_left += 1 << 20;
            same(&m, want, get(&m));
        } else if (!strcmp(s, "capture")) {
            capturing = 1;  /* on another stream, in another thread's global mode */
            drop(&m);
            capturing = 0;
            if (refused || pinned_live) fail("pinned memory lost when a case goes during a capture");
            free(want);
            continue;
        } else {
            fail("no such scenario");
        }
        free(want);
        drop(&m);
        if (pinned_live) fail("pinned memory left");
    }
    printf("ok\n");
    return 0;
}
