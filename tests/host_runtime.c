/*
 * Host-side runs of the library against a stand-in for the HIP runtime
 * (tests/test_host_runtime.py builds this program, links it to libxfft.so and
 * runs it on the CPU; no GPU is used).  The functions below take the place of
 * the runtime's: device memory is zero-initialised host memory, kernels are
 * counted and not run, and what the host code reads back from them (list
 * lengths of the setup) or from the runtime (event times) is scripted.  What a
 * scenario checks is host code only: which launches, allocations, waits and
 * attributes the library asks for.
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "xfft.h"

typedef struct { uint32_t x, y, z; } Dim3;

/* ---------------------------------------------------------------- scripted state */
static int64_t g_totals[3];             /* irregular voxels, enriched nodes, cut elements */
static int g_scans;                     /* scans since the last setup */
static unsigned g_reg_grid;             /* workgroups of the last regular-voxel launch */
static int g_last_regular;              /* the last launch was an operator application */
static float (*g_elapsed)(void);        /* event time of the launches since the last one, < 0: the call fails */
static int g_timings;
static int g_mallocs, g_frees, g_waits, g_launches;
static int g_device, g_big_launches, g_bad_launches;   /* current device; launches above 64 KB of dynamic LDS */

/* ---------------------------------------------------------------- kernels */
static struct { const void *f; char name[512]; size_t lds[2]; } g_kernels[4096];
static int g_nkernels;
static void *g_module;

void **__hipRegisterFatBinary(const void *data) { (void)data; return &g_module; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *var, char *hv, char *dv, int ext, size_t size, int c, int g) {
    (void)m; (void)var; (void)hv; (void)dv; (void)ext; (void)size; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned t, void *a, void *b, void *c,
                           void *d, int *w) {
    (void)m; (void)df; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (g_nkernels == 4096) { fprintf(stderr, "too many kernels\n"); exit(2); }
    g_kernels[g_nkernels].f = f;
    snprintf(g_kernels[g_nkernels++].name, 512, "%s", name);
}
static int kernel_index(const void *f) {
    for (int i = 0; i < g_nkernels; ++i)
        if (g_kernels[i].f == f) return i;
    fprintf(stderr, "kernel not registered\n");
    exit(2);
}

static struct { Dim3 g, b; size_t lds; void *s; } g_cfg;
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void *s) {
    g_cfg.g = g; g_cfg.b = b; g_cfg.lds = lds; g_cfg.s = s;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **s) {
    *g = g_cfg.g; *b = g_cfg.b; *lds = g_cfg.lds; *s = g_cfg.s;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **args, size_t lds, void *s) {
    (void)block; (void)s;
    ++g_launches;
    const int k = kernel_index(f);
    const char *n = g_kernels[k].name;
    if (lds > 65536) {
        ++g_big_launches;
        if (g_kernels[k].lds[g_device] < lds) {
            if (!g_bad_launches++) fprintf(stderr, "%s: %zu bytes of LDS on device %d\n", n, lds, g_device);
        }
    }
    g_last_regular = 0;
    if (strstr(n, "k_regular")) { g_reg_grid = grid.x; g_last_regular = 1; }
    if (strstr(n, "k_scan_offsets")) **(int64_t **)args[3] = g_totals[g_scans++ % 3];
    if (strstr(n, "k_classify")) **(unsigned long long **)args[9] = (unsigned long long)g_totals[2];
    return 0;
}
int hipGetLastError(void) { return 0; }

/* ---------------------------------------------------------------- devices, memory, streams, events */
int hipGetDeviceCount(int *n) { *n = 2; return 0; }
int hipSetDevice(int d) { g_device = d; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)a; g_kernels[kernel_index(f)].lds[g_device] = (size_t)v; return 0; }
int hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = calloc(1, (size_t)64 << 20); return *p ? 0 : 2; }
int hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)288 << 30; return 0; }
int hipMalloc(void **p, size_t n) { ++g_mallocs; *p = calloc(1, n ? n : 1); return *p ? 0 : 2; }
int hipFree(void *p) { ++g_frees; free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return hipMalloc(p, n); }
int hipHostFree(void *p) { return hipFree(p); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *q) { (void)k; (void)q; memcpy(d, s, n); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *q) { (void)q; memset(d, v, n); return 0; }
int hipStreamCreate(void **s) { return hipMalloc(s, 1); }
int hipStreamDestroy(void *s) { return hipFree(s); }
int hipStreamSynchronize(void *s) { ++g_waits; (void)s; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipEventCreate(void **e) { return hipMalloc(e, 1); }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipMalloc(e, 1); }
int hipEventDestroy(void *e) { return hipFree(e); }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) {
    (void)a; (void)b;
    *ms = 1.0f;
    if (!g_last_regular || !g_elapsed) return 0;
    ++g_timings;
    *ms = g_elapsed();
    return *ms < 0.0f ? 1 : 0;
}

/* ---------------------------------------------------------------- problems */
static int g_checks, g_fail;
static void expect(int got, int want, const char *what) {
    ++g_checks;
    if (got != want) {
        ++g_fail;
        fprintf(stderr, "FAIL %s: got %d, want %d\n", what, got, want);
    }
}

static xfft_problem *make_problem(int n0, int n1, int n2, int device, int precision) {
    const int32_t n[3] = {n0, n1, n2};
    const double len[3] = {n0, n1, n2}, lame[4] = {0.5, 0.4, 5.0, 4.0};
    const size_t N = (size_t)n0 * n1 * n2;
    double *L = malloc(sizeof(double) * N);
    int32_t *ph = calloc(N, sizeof(int32_t));
    for (size_t i = 0; i < N; ++i) L[i] = 1.0;
    xfft_options o;
    xfft_default_options(&o);
    o.device = device;
    o.precision = precision;
    xfft_problem *p = NULL;
    g_scans = 0;
    expect(xfft_setup(n, len, L, ph, 2, lame, &o, &p), XFFT_OK, "setup");
    free(L);
    free(ph);
    return p;
}

/* ---------------------------------------------------------------- depth of the regular-voxel march
 * 128 x 128 x 32 has 9 x 9 tiles; the default depth is 8 planes (4 chunks).  Timings of
 * the depths 4, 8, 16, 32 per round: t[round][depth index]. */
enum { TILES = 81, N2 = 32 };
static float g_t[2][4];
static int g_fail_at, g_seen[4];
static float depth_time(void) {
    const int depth = N2 / (int)(g_reg_grid / TILES), c = depth == 4 ? 0 : depth == 8 ? 1 : depth == 16 ? 2 : 3;
    if (g_timings == g_fail_at) return -1.0f;
    const int round = g_seen[c]++ ? 1 : 0;
    return g_t[round][c];
}
static int depth_of_solve(int n0, const float t[2][4], int fail_at) {
    memcpy(g_t, t, sizeof(g_t));
    memset(g_seen, 0, sizeof(g_seen));
    g_timings = 0;
    g_fail_at = fail_at;
    const double e[6] = {1, 0, 0, 0, 0, 0};
    double avg[6];
    xfft_problem *p = make_problem(n0, 256 - n0, N2, 0, XFFT_FP64);
    const int rc = xfft_solve(p, 1, e, NULL, NULL, avg, NULL, NULL);
    expect(rc >= 0, 1, "solve");
    xfft_destroy(p);
    return N2 / (int)(g_reg_grid / TILES);
}
static void scenario_depth(const char *which) {
    /* one case per process: results are kept per grid */
    g_elapsed = depth_time;
    if (!strcmp(which, "close")) {               /* 1 % ahead in both rounds: within the noise */
        const float t[2][4] = {{1.2f, 1.0f, 0.99f, 1.1f}, {1.2f, 1.0f, 0.99f, 1.1f}};
        expect(depth_of_solve(128, t, 0), 8, "depth 1 % faster is not taken");
    } else if (!strcmp(which, "outlier")) {      /* the default's first timing was disturbed */
        const float t[2][4] = {{1.2f, 1.1f, 1.02f, 1.2f}, {1.2f, 1.0f, 1.02f, 1.1f}};
        expect(depth_of_solve(128, t, 0), 8, "a disturbed timing does not decide");
    } else if (!strcmp(which, "faster")) {       /* and a depth that pays is taken, once per grid */
        const float t[2][4] = {{1.2f, 1.0f, 0.96f, 0.97f}, {1.2f, 1.0f, 0.95f, 0.97f}};
        expect(depth_of_solve(128, t, 0), 16, "depth 5 % faster is taken");
        const float u[2][4] = {{9, 9, 9, 9}, {9, 9, 9, 9}};
        expect(depth_of_solve(128, u, 0), 16, "depth kept for the grid");
        expect(g_timings, 0, "no timing for a known grid");
    } else {                                     /* a failed timing: default, and nothing kept */
        const float t[2][4] = {{0.5f, 1.0f, 0.9f, 1.2f}, {0.5f, 1.0f, 0.9f, 1.2f}};
        expect(depth_of_solve(128, t, 3), 8, "default depth after a failed timing");
        const float u[2][4] = {{1.2f, 1.0f, 0.9f, 1.2f}, {1.2f, 1.0f, 0.9f, 1.2f}};
        expect(depth_of_solve(128, u, 0), 16, "timed again by the next problem");
    }
}

/* ---------------------------------------------------------------- dynamic LDS on a second device
 * Every launch above 64 KB needs the kernel's attribute on the device it runs on. */
static void scenario_devices(int n, int precision) {
    g_totals[0] = 100; g_totals[1] = 300; g_totals[2] = 400;
    for (int dev = 0; dev < 2; ++dev) {
        xfft_problem *p = make_problem(n, n, 16, dev, precision);
        const size_t ndof = 3 * ((size_t)n * n * 16 + 300);
        double *x = calloc(ndof, sizeof(double)), *y = calloc(ndof, sizeof(double)), avg[36], res2;
        double e[36] = {0};
        for (int k = 0; k < 6; ++k) e[7 * k] = 1.0;
        const int before = g_big_launches;
        expect(xfft_apply_operator_noalloc(p, x, e, y, avg, NULL), XFFT_OK, "noalloc operator");
        expect(xfft_apply_operator_noalloc(p, x, NULL, y, NULL, NULL), XFFT_OK, "noalloc operator");
        for (int prec = XFFT_FP64; prec <= XFFT_FP32; prec += 2) {
            expect(xfft_apply_operator(p, prec, x, e, y, avg), XFFT_OK, "operator");
            expect(xfft_apply_precond(p, prec, x, y, &res2), XFFT_OK, "preconditioner");
        }
        expect(xfft_solve(p, 6, e, NULL, NULL, avg, NULL, NULL) >= 0, 1, "solve");
        expect(g_big_launches > before, 1, "launches above 64 KB");
        expect(g_bad_launches, 0, "launches without the attribute on their device");
        free(x);
        free(y);
        xfft_destroy(p);
    }
}

/* ---------------------------------------------------------------- cost of building a problem
 * Small grids pay for the calls of the setup, not for its kernels: allocations and
 * waits of xfft_setup, and frees of the scratch it takes, at most those given. */
static void scenario_setup(int n0, int n1, int mallocs, int frees, int waits) {
    g_totals[0] = 100; g_totals[1] = 300; g_totals[2] = 400;
    make_problem(16, 16, 16, 0, XFFT_FP64);              /* first use of the device */
    g_mallocs = g_frees = g_waits = g_launches = 0;
    xfft_problem *p = make_problem(n0, n1, 12, 0, XFFT_FP64);
    printf("%d allocations, %d frees, %d waits, %d launches\n", g_mallocs, g_frees, g_waits, g_launches);
    expect(g_mallocs <= mallocs, 1, "allocations of a setup");
    expect(g_frees <= frees, 1, "frees of a setup");
    expect(g_waits <= waits, 1, "waits of a setup");
    xfft_destroy(p);
    expect(g_mallocs, g_frees, "everything freed with the problem");
}

int main(int argc, char **argv) {
    if (argc == 7 && !strcmp(argv[1], "setup"))
        scenario_setup(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]));
    else if (argc == 4 && !strcmp(argv[1], "devices")) scenario_devices(atoi(argv[2]), atoi(argv[3]));
    else if (argc == 3 && !strcmp(argv[1], "depth")) scenario_depth(argv[2]);
    else return 2;
    if (g_fail) return 1;
    printf("host_runtime: %d checks passed\n", g_checks);
    return 0;
}
