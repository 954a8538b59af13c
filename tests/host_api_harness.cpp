// The host side of the C ABI (vg_api.cpp) without a GPU: the HIP calls and the
// kernel launchers are stand-ins that only count, fail on demand or check what
// they are given.  Built and run by test_host_api.py, one scenario per run.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>

#include "vg_internal.h"

static int g_launches = 0, g_fail_at = -1;   // launches so far; the one that fails
static bool g_band = false, g_no_alloc = false;

void *operator new(std::size_t n) {
    if (g_no_alloc) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

static int launch() { return g_launches++ == g_fail_at ? VG_EHIP : VG_OK; }

extern "C" {
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *b, const void *, int, size_t) {
    *b = 8;
    return hipSuccess;
}
int vg_rank_bytes(int, int, int, int, size_t *b) { *b = 0; return VG_OK; }
}

namespace vg {
int make_geom(int nx, int ny, int nz, int b, Geom *g) {
    *g = Geom{nx, ny, nz, b, 0, 0, 0, (int64_t)nx * ny * nz, 0};
    return VG_OK;
}
int launch_pass2(vg_sim *h, int mode, int, double, double, hipStream_t, const TileRange *) {
    if (h->band_mid && mode != MODE_DT) {
        std::printf("a pass of mode %d reads the second field set\n", mode);
        std::exit(1);
    }
    const int rc = launch();
    if (rc) return rc;
    if (h->band_mid) h->band_mid = 0;
    else if (mode == MODE_D || mode == MODE_DT) h->cur ^= 1;
    return VG_OK;
}
int launch_pass(vg_sim *h, int mode, int tot, double dt, hipStream_t s) {
    return launch_pass2(h, mode, tot, dt, dt, s, nullptr);
}
int launch_pass_bufs(vg_sim *, int, int, double, const void *const *, void *const *, hipStream_t, void *) {
    return launch();
}
int launch_band_pair(vg_sim *h, double, hipStream_t) {
    const int rc = launch();
    if (!rc) h->band_mid ^= 1;
    return rc;
}
int launch_totals_finalize(vg_sim *, double *, int, hipStream_t) { return VG_OK; }
int launch_geometry(vg_sim *, hipStream_t) { return VG_OK; }
bool use_rank(const vg_sim *) { return false; }
bool use_offsets(const vg_sim *) { return false; }
bool use_relative(const vg_sim *) { return true; }
bool band_geometry(const vg_sim *) { return false; }
bool use_band(const vg_sim *) { return g_band; }
bool tape_keeps_dom(const vg_sim *) { return false; }
int tape_rows(const vg_sim *) { return VG_NPOOL; }
void tape_pass_bufs(const vg_sim *, void *, int64_t, const void **, void **, void **) {}
int build_band(vg_sim *, hipStream_t) { return VG_OK; }
int build_offsets(vg_sim *, hipStream_t) { return VG_OK; }
PackedNbr packed_of(const vg_sim *) { return PackedNbr{}; }
int restore_canonical(vg_sim *h, hipStream_t) { h->cur = 0; return VG_OK; }
int run_cg(vg_sim *, int, double, double, int, int *, double *, hipStream_t) { return VG_OK; }
void mg_plan(vg_sim *) {}
int mg_build(vg_sim *, hipStream_t) { return VG_OK; }
int mg_apply(vg_sim *, double, const double *, double *, hipStream_t) { return VG_OK; }
int launch_record(vg_sim *, int64_t, double, void *, hipStream_t) { return VG_OK; }
int launch_adjoint(vg_sim *, int64_t, double, const void *, const double *, void *, double *, hipStream_t) {
    return VG_OK;
}
int launch_seed(vg_sim *, const double *, void *, int, hipStream_t) { return VG_OK; }
int launch_load_state(vg_sim *, const void *, int, hipStream_t) { return VG_OK; }
int launch_store_state(vg_sim *, void *, int, hipStream_t) { return VG_OK; }
}  // namespace vg

static void need(bool ok, const char *what) {
    if (ok) return;
    std::printf("failed: %s\n", what);
    std::exit(1);
}

static vg_sim *make(int64_t n, int prec) {
    static int64_t seg[2];
    seg[0] = 0;
    seg[1] = n;
    vg_desc d{};
    d.n = n;
    d.nseg = 1;
    d.precision = prec;
    d.seg_off = seg;
    d.nbr_d = (const int32_t *)0x1000;
    vg_sim *h = nullptr;
    need(vg_create(&d, &h) == VG_OK, "vg_create");
    return h;
}

static void bind(vg_sim *h, char *work, size_t bytes) {
    need(vg_init_state(h, work, work, work, bytes, nullptr) == VG_OK, "vg_init_state");
}

// A run that fails at any of its launches leaves later passes on the bound fields.
static void failed_runs() {
    g_band = true;
    vg_sim *h = make(1000, VG_F64);
    size_t bytes = 0;
    vg_workspace_bytes(h, &bytes);
    char *work = (char *)std::calloc(1, bytes + 64);
    bind(h, work, bytes);
    vg_set_launch_options(h, VG_LAUNCH_GRAPHS_OFF);
    vg_params p = h->params;
    for (int order : {VG_ORDER_TD, VG_ORDER_DT}) {
        p.step_order = order;
        need(vg_set_params(h, &p) == VG_OK, "vg_set_params");
        bool ended = false;
        for (int fail = 0; !ended; fail++) {
            bind(h, work, bytes);
            g_launches = 0;
            g_fail_at = fail;
            const int rc = vg_step_explicit(h, 12, 0.01, 0, nullptr, VG_FORCE, nullptr);
            need(rc == (fail < g_launches ? VG_EHIP : VG_OK), "status of the run");
            ended = rc == VG_OK;
            need(h->band_mid == 0, "the run leaves the state in the second set");
            g_fail_at = -1;
            need(vg_step_subcycled(h, 2, 0.01, 0.005, VG_FORCE, nullptr) == VG_OK, "sub-cycled step");
        }
        h->band_mid = 1;
        bind(h, work, bytes);
        need(h->band_mid == 0, "binding new buffers");
    }
}

// A step of compensated fields large enough for slabs allocates nothing: an
// exception must not leave the C entry.
static void no_allocation() {
    vg_sim *h = make(8000000, VG_F32C);
    size_t bytes = 0;
    vg_workspace_bytes(h, &bytes);
    char *work = (char *)std::calloc(1, bytes);
    need(work != nullptr, "workspace");
    bind(h, work, bytes);
    h->xy_dist = 200;
    h->z_dist = 10000;
    std::vector<double> log(40 * 6);
    for (int order : {VG_ORDER_TD, VG_ORDER_DT}) {
        vg_params p = h->params;
        p.step_order = order;
        need(vg_set_params(h, &p) == VG_OK, "vg_set_params");
        g_launches = 0;
        g_no_alloc = true;
        const int rc = vg_step_explicit(h, 37, 0.01, 3, log.data(), VG_FORCE, nullptr);
        g_no_alloc = false;
        need(rc == VG_OK, "step");
        need(g_launches > 38, "the passes ran slab by slab");
    }
}

// Runs of fewer than four passes gain nothing from slabs: one launch a pass;
// so do fields little larger than the last-level cache.
static void short_runs() {
    struct Run {
        int64_t n, steps, launches;   // launches 0: slab by slab
    };
    for (const Run &r : {Run{8000000, 1, 2}, Run{8000000, 2, 3}, Run{8000000, 3, 0}, Run{7000000, 12, 13}}) {
        vg_sim *h = make(r.n, VG_F32C);
        size_t bytes = 0;
        vg_workspace_bytes(h, &bytes);
        char *work = (char *)std::calloc(1, bytes);
        need(work != nullptr, "workspace");
        bind(h, work, bytes);
        h->xy_dist = 200;
        h->z_dist = 10000;
        g_launches = 0;
        need(vg_step_explicit(h, r.steps, 0.01, 0, nullptr, VG_FORCE, nullptr) == VG_OK, "step");
        need(r.launches ? g_launches == r.launches : g_launches > r.steps + 1, "launches of the run");
        vg_destroy(h);
        std::free(work);
    }
}

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "failed_runs") failed_runs();
    else if (what == "no_allocation") no_allocation();
    else if (what == "short_runs") short_runs();
    else need(false, "scenario name");
    std::printf("ok\n");
    return 0;
}
