/* libpt's host code over a HIP runtime without a device: this program defines the HIP calls that the
 * library makes (its own definitions come before the runtime's), counts them, and limits the memory they
 * hand out.  Device memory is host memory that no kernel touches; kernels are counted and not run.
 *
 *   fake_hip <scenario>     prints what failed and exits 1, or prints "ok" and exits 0
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "pt.h"

/* ---- the runtime ------------------------------------------------------------------------- */
enum { SUCCESS = 0, INVALID = 1, OUT_OF_MEMORY = 2, CAPTURE_IMPLICIT = 906 };
typedef struct { unsigned x, y, z; } dim3_;

#define MAX_BLOCKS 4096
static struct { void* p; size_t bytes; int device; } blocks[MAX_BLOCKS];
static size_t live[2], limit[2] = {(size_t)1 << 40, (size_t)1 << 40};
static int nlive[2], mallocs, frees, launches, device, capture_query, last_error;

static int give(int e) {
    if (e) last_error = e;
    return e;
}
int hipGetDeviceCount(int* n) { *n = 2; return SUCCESS; }
int hipGetDevice(int* d) { *d = device; return SUCCESS; }
int hipSetDevice(int d) { device = d; return SUCCESS; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return SUCCESS; }
int hipDeviceSynchronize(void) { return SUCCESS; }
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }
int hipMalloc(void** p, size_t bytes) {
    ++mallocs;
    *p = NULL;
    if (live[device] + bytes > limit[device]) return give(OUT_OF_MEMORY);
    for (int q = 0; q < MAX_BLOCKS; ++q)
        if (!blocks[q].p) {
            blocks[q].p = *p = malloc(bytes);
            blocks[q].bytes = bytes;
            blocks[q].device = device;
            live[device] += bytes;
            ++nlive[device];
            return SUCCESS;
        }
    return give(INVALID);
}
int hipFree(void* p) {
    ++frees;
    for (int q = 0; q < MAX_BLOCKS; ++q)
        if (p && blocks[q].p == p) {
            live[blocks[q].device] -= blocks[q].bytes;
            --nlive[blocks[q].device];
            blocks[q].p = NULL;
            free(p);
            return SUCCESS;
        }
    fprintf(stderr, "free of %p, which is not live\n", p);
    exit(1);
}
int hipHostMalloc(void** p, size_t bytes, unsigned f) { (void)f; *p = calloc(1, bytes); return SUCCESS; }
int hipHostFree(void* p) { free(p); return SUCCESS; }
int hipMemcpyAsync(void* d, const void* s, size_t bytes, int kind, void* st) {
    (void)st;
    if (kind == 2) memcpy(d, s, bytes);   /* device to host: the error words of a load */
    return SUCCESS;
}
int hipMemsetAsync(void* d, int v, size_t bytes, void* st) { (void)st; memset(d, v, bytes); return SUCCESS; }
int hipStreamSynchronize(void* s) { (void)s; return SUCCESS; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = 0; return give(capture_query); }
int hipEventCreate(void** e) { *e = malloc(1); return SUCCESS; }
int hipEventDestroy(void* e) { free(e); return SUCCESS; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return SUCCESS; }
int hipEventSynchronize(void* e) { (void)e; return SUCCESS; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.0f; return SUCCESS; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l) {
    (void)f; (void)b; (void)l;
    *n = 2;
    return SUCCESS;
}
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** a, size_t l, void* s) {
    (void)f; (void)g; (void)b; (void)a; (void)l; (void)s;
    ++launches;
    return SUCCESS;
}

/* ---- helpers ------------------------------------------------------------------------------ */
static int failures;
#define CHECK(cond, ...)                                  \
    do {                                                  \
        if (!(cond)) {                                    \
            printf("%s:%d: ", __func__, __LINE__);        \
            printf(__VA_ARGS__);                          \
            printf("\n");                                 \
            ++failures;                                   \
        }                                                 \
    } while (0)

/* A grid of nx x 1 x 1 cells loaded from device arrays (whose contents no one reads). */
static pt_grid* load(int nx) {
    static char somewhere[8];
    pt_grid_desc d;
    memset(&d, 0, sizeof d);
    d.nx = nx;
    d.ny = d.nz = 1;
    d.dx = d.dy = d.dz = 1.0;
    d.qx = d.qy = d.qz = (const double*)somewhere;
    d.flags = (const int32_t*)somewhere;
    d.porosity_scalar = 0.3;
    d.mem = PT_MEM_DEVICE;
    d.balance_tol = -1.0;
    pt_grid* g = NULL;
    int rc = pt_load_grid(&d, NULL, &g);
    CHECK(rc == PT_OK, "load of %d cells: %d (%s)", nx, rc, pt_last_error());
    return g;
}
static size_t bytes_of(int nx) {   /* device memory of such a grid */
    size_t before = live[device];
    pt_grid* g = load(nx);
    size_t b = live[device] - before;
    pt_release(g);
    pt_shutdown();
    return b;
}

enum { PLAIN, SORTED, SERIES, COUNT, KINDS };   /* calls with different buffers */
static int track(pt_grid* g, int kind, int64_t n) {
    static char somewhere[8];
    static const double snaps[2] = {1.0, 2.0};
    pt_particles p;
    pt_track_opts o;
    memset(&p, 0, sizeof p);
    p.n = n;
    p.cell = p.status = p.ncross = (int32_t*)somewhere;
    p.xi = p.eta = p.zeta = p.t = (double*)somewhere;
    p.path_hash = (uint64_t*)somewhere;
    pt_default_opts(&o);
    o.sort = kind == SORTED ? PT_SORT_CELL : PT_SORT_NONE;
    if (kind == SERIES) {
        o.mode = PT_TIMESERIES;
        o.snap_times = snaps;
        o.n_snap = 2;
        o.snap_xyz = (double*)somewhere;
    }
    if (kind == COUNT) {
        o.mode = PT_PATHLINE;
        o.path_count_only = 1;
        o.path_offsets = (int64_t*)somewhere;
    }
    const pt_grid* gs[1] = {g};
    pt_run* r = NULL;
    int rc = pt_track(gs, 1, &p, &o, NULL, &r);
    if (rc == PT_OK) {
        pt_summary s;
        CHECK(pt_results(r, &s) == PT_OK, "results: %s", pt_last_error());
        pt_release(r);
    }
    return rc;
}

/* ---- scenarios ---------------------------------------------------------------------------- */

/* A call whose run buffers fit only in the memory of a grid that was released before it; the sizes of
 * that grid let every allocation of the call be the first without memory. */
static void run_buffers(void) {
    for (int kind = 0; kind < KINDS; ++kind) {
        const int64_t n = 1 << 20;
        pt_grid* a = load(1000);
        const size_t grid = live[0];
        CHECK(track(a, kind, n) == PT_OK, "kind %d without a limit: %s", kind, pt_last_error());
        const size_t run = live[0] - grid;
        pt_release(a);
        pt_shutdown();
        for (int nx = 2100; nx < 400000; nx = nx * 3 / 2) {
            a = load(1000);
            pt_release(load(nx));
            limit[0] = live[0] > grid + run ? live[0] : grid + run;   /* no room for anything else */
            CHECK(track(a, kind, n) == PT_OK, "kind %d beside a released grid of %d: %s", kind, nx, pt_last_error());
            CHECK(live[0] == grid + run, "kind %d beside a released grid of %d: %zu bytes live, %zu used", kind, nx, live[0], grid + run);
            limit[0] = (size_t)1 << 40;
            pt_release(a);
            pt_shutdown();
        }
    }
    /* an allocation that does not fit at all is refused, and the next call runs */
    pt_grid* a = load(1000);
    pt_release(load(3000));
    limit[0] = live[0] + 1024;
    CHECK(track(a, SORTED, 1 << 20) == PT_ERR_OOM, "refusal");
    CHECK(nlive[0] <= 2, "%d blocks kept after a refusal", nlive[0]);
    limit[0] = (size_t)1 << 40;
    CHECK(track(a, SORTED, 1 << 20) == PT_OK, "after a refusal: %s", pt_last_error());
    pt_release(a);
}

/* A grid's memory is taken again by a load of about its size, and by that only. */
static void reuse(void) {
    const size_t b = bytes_of(1000);
    pt_grid* g = load(1000);
    pt_release(g);
    int m = mallocs, f = frees;
    for (int q = 0; q < 20; ++q) pt_release(load(1000 - q));
    CHECK(mallocs == m && frees == f, "%d allocations and %d frees in a loop over one size", mallocs - m, frees - f);
    CHECK(live[0] == b, "%zu bytes live, one grid takes %zu", live[0], b);
    g = load(400);   /* less than half */
    CHECK(mallocs == m + 1, "a block of more than twice the size was taken");
    pt_grid* h = load(1100);
    CHECK(mallocs == m + 2, "a block too small was taken");
    pt_release(g);
    pt_release(h);
    pt_shutdown();
    CHECK(live[0] == 0 && nlive[0] == 0, "%zu bytes live after the shutdown", live[0]);
}

/* The limits are a device's own; the oldest blocks leave first. */
static void limits(void) {
    const int max_blocks = 8;
    const size_t max_bytes = (size_t)256 << 20;
    pt_grid* g[20];
    for (int q = 0; q < 20; ++q) g[q] = load(1000 * (q + 1));
    const int in_use = nlive[0];
    CHECK(in_use == 20, "%d blocks for 20 grids", in_use);
    for (int q = 0; q < 20; ++q) pt_release(g[q]);
    CHECK(nlive[0] == max_blocks, "%d blocks kept", nlive[0]);
    /* a loop over a size that the full pool does not hold finds its own block the second time */
    pt_release(load(100000));
    int m = mallocs;
    for (int q = 0; q < 5; ++q) pt_release(load(100000));
    CHECK(mallocs == m, "%d allocations in a loop over a new size", mallocs - m);
    CHECK(nlive[0] == max_blocks, "%d blocks kept", nlive[0]);
    /* the other device has room of its own */
    device = 1;
    for (int q = 0; q < 8; ++q) g[q] = load(1000);
    for (int q = 0; q < 8; ++q) pt_release(g[q]);
    CHECK(nlive[0] == max_blocks && nlive[1] == max_blocks, "%d and %d blocks kept", nlive[0], nlive[1]);
    m = mallocs;
    for (int q = 0; q < 8; ++q) g[q] = load(1000);
    CHECK(mallocs == m, "blocks of the device were not taken");
    for (int q = 0; q < 8; ++q) pt_release(g[q]);
    device = 0;
    /* bytes: 100 MB grids, and one above the limit, which leaves the others alone */
    const int n100 = 100 * 1000 * 1000 / 124;
    for (int q = 0; q < 4; ++q) g[q] = load(n100);
    for (int q = 0; q < 4; ++q) pt_release(g[q]);
    CHECK(live[0] <= max_bytes && live[0] > max_bytes / 2, "%zu bytes kept", live[0]);
    const size_t kept = live[0];
    pt_release(load(3 * n100));
    CHECK(live[0] == kept, "%zu bytes kept, %zu before", live[0], kept);
    pt_shutdown();
    CHECK(live[0] == 0 && live[1] == 0, "%zu and %zu bytes live after the shutdown", live[0], live[1]);
}

/* The default stream while another stream is being captured: the runtime refuses to say whether it is
 * being captured.  The call runs, and does not rely on what an uncertain call left behind. */
static void capture_refused(void) {
    pt_grid* g = load(1000);
    int n = launches;
    CHECK(track(g, PLAIN, 1000) == PT_OK, "%s", pt_last_error());
    const int first = launches - n;
    n = launches;
    CHECK(track(g, PLAIN, 1000) == PT_OK, "%s", pt_last_error());
    CHECK(launches - n == first - 1, "%d kernels, %d in the first call", launches - n, first);   /* no reset */
    pt_release(g);
    pt_shutdown();
    g = load(1000);
    capture_query = CAPTURE_IMPLICIT;
    for (int q = 0; q < 3; ++q) CHECK(track(g, PLAIN, 1000) == PT_OK, "call %d: %s", q, pt_last_error());
    CHECK(last_error == 0, "the refusal was left behind as error %d", last_error);
    capture_query = 0;
    pt_release(g);
}

int main(int argc, char** argv) {
    const char* s = argc > 1 ? argv[1] : "";
    if (!strcmp(s, "run_buffers")) run_buffers();
    else if (!strcmp(s, "reuse")) reuse();
    else if (!strcmp(s, "limits")) limits();
    else if (!strcmp(s, "capture_refused")) capture_refused();
    else return 2;
    pt_shutdown();
    if (live[0] || live[1]) {
        printf("%zu and %zu bytes live at the end\n", live[0], live[1]);
        ++failures;
    }
    if (!failures) printf("ok\n");
    return failures ? 1 : 0;
}
