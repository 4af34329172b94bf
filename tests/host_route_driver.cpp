// Driver for the dispatch of the C-ABI library on the CPU: the library's host
// source linked against a stand-in of the HIP runtime and of the kernel
// launchers.  The stand-in copies host memory, keeps a clock per launch (so
// the tuner measures the times a scenario sets), orders streams, events and
// graphs, and logs what was launched; it reports a graph that is destroyed or
// changed while work that uses it may still run.  Scenario by name; prints OK
// or what went wrong.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "fuglbm.h"
#include "kernels.h"

// ---- what happened -------------------------------------------------------
static int failures = 0;
static void fault(const std::string &what) {
    std::printf("%s\n", what.c_str());
    ++failures;
}
#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) fault(std::string(__func__) + ": not " #c + " (line " +     \
                        std::to_string(__LINE__) + ")");                      \
    } while (0)

static double now_ms = 0.0;                  // the device's clock
static std::map<std::string, int> launched;  // by kernel
static std::map<std::string, double> cost;   // ms of a launch, by kernel
static int captures = 0, pinned_calls = 0;
static size_t pinned_bytes = 0;
static int lane_launches = 0;                // launches on streams of the library
static hipStream_t user_stream = nullptr;

// ---- streams, events, graphs ---------------------------------------------
using Clock = std::map<const void *, long>;  // stream -> work items known done before
struct Graph {
    std::vector<std::string> nodes;
};
struct Exec {
    std::vector<std::string> nodes;
    Clock used;                              // stream -> last launch of it there
    bool alive = true;
};
struct Event {
    Clock at;
    double ms = 0.0;
};
struct Stream {
    long seq = 0;
    Clock seen;
    Graph *capture = nullptr;
};
static std::map<const void *, Stream> streams;
static Clock host_seen;
static void merge(Clock &a, const Clock &b) {
    for (auto &k : b) a[k.first] = std::max(a[k.first], k.second);
}
static Clock clock_of(const void *s) {
    Clock c = streams[s].seen;
    c[s] = streams[s].seq;
    return c;
}
static void run(const std::string &kernel, const void *st) {
    Stream &s = streams[st];
    if (s.capture) {
        s.capture->nodes.push_back(kernel);
        return;
    }
    ++s.seq;
    if (st != user_stream) ++lane_launches;
    ++launched[kernel];
    auto it = cost.find(kernel);
    now_ms += it == cost.end() ? 0.001 : it->second;
}
static bool in_flight(const Clock &used) {
    for (auto &k : used)
        if (host_seen[k.first] < k.second) return true;
    return false;
}

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipMalloc(void **p, size_t n) {
    *p = std::calloc(n ? n : 1, 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    ++pinned_calls;
    pinned_bytes += n;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    if (streams[s].capture) return hipErrorStreamCaptureUnsupported;
    merge(host_seen, clock_of(s));
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = (hipEvent_t) new Event();
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    ((Event *)e)->at = clock_of(s);
    ((Event *)e)->ms = now_ms;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    merge(host_seen, ((Event *)e)->at);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(((Event *)b)->ms - ((Event *)a)->ms);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    merge(streams[s].seen, ((Event *)e)->at);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    ++captures;
    streams[s].capture = new Graph();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
    *g = (hipGraph_t)streams[s].capture;
    streams[s].capture = nullptr;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
    *c = streams[s].capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    auto *e = new Exec();
    e->nodes = ((Graph *)g)->nodes;
    *x = (hipGraphExec_t)e;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph *)g; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st) {
    auto *e = (Exec *)x;
    if (!e->alive) fault("a destroyed graph was launched");
    if (streams[st].capture) return hipErrorStreamCaptureUnsupported;
    for (auto &k : e->nodes) run(k, st);
    e->used[st] = streams[st].seq;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    auto *e = (Exec *)x;
    if (!e->alive) fault("a graph was destroyed twice");
    if (in_flight(e->used)) fault("a graph was destroyed while it may still run");
    e->alive = false;          // kept, so that a later use shows
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static char mem[1 << 24];
    *p = mem;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *,
                           void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t st) {
    run("noalloc tables", st);
    return hipSuccess;
}
int roctxRangePushA(const char *) { return 0; }
int roctxRangePop() { return 0; }
}

// ---- the kernels' launchers -------------------------------------------------
// last arguments seen
static int last_rows = 0, last_members = 0, stream3_items = 0, stream3_waves = 0;
static Tiles3 stream3_tiles;

hipError_t launch_init(int, bool, const SimConst *, int64_t, const double *, void *, hipStream_t s) {
    run("init", s);
    return hipSuccess;
}
hipError_t launch_step_generic(int, bool, const SimConst *, int, int, int, int, const void *, void *,
                               double *, double *, double *, double *, double *, uint32_t *, bool,
                               hipStream_t s) {
    run("passes", s);
    return hipSuccess;
}
hipError_t launch_planes(int, bool, bool, int, int, int, int, int, int, void *, void *,
                         hipStream_t s) {
    run("planes", s);
    return hipSuccess;
}
hipError_t launch_to_host(const double *a, int64_t na, const double *b, int64_t nb,
                          const uint32_t *status, double *to, uint32_t *word, hipStream_t s) {
    run("to_host", s);
    if (na) std::memcpy(to, a, na * 8);
    if (nb) std::memcpy(to + na, b, nb * 8);
    *word = *status;
    return hipSuccess;
}
// tiles of 16 x 4 x 4 and 64 x 2 x 2 sites
void generic_units(int, int ncomp, int nx, int ny, int nz, int64_t units[3]) {
    auto up = [](int a, int b) { return (int64_t)((a + b - 1) / b); };
    units[0] = ((int64_t)nx * ny * nz + 255) / 256;
    units[1] = up(nx, 16) * up(ny, 4) * up(nz, 4);
    units[2] = up(nx, 64) * up(ny, 2) * up(nz, 2) * ncomp;
}
hipError_t launch_step_generic_batch(int, bool, bool, const GenMember *, int n, const int64_t[3], int,
                                     hipStream_t s) {
    last_members = n;
    run("passes batch", s);
    return hipSuccess;
}
hipError_t launch_fields(int, bool, const SimConst *, int, int, int, const void *, double *, double *,
                         double *, double *, double *, uint32_t *, hipStream_t s) {
    run("fields", s);
    return hipSuccess;
}
hipError_t launch_diag(int, int, int64_t, const double *, const double *, const double *, double *,
                       double *, int, double *, int, hipStream_t s) {
    run("diag", s);
    return hipSuccess;
}
int diag_blocks(int64_t) { return 1; }
int fused_blocks_per_cu(int, bool) { return 2; }
hipError_t launch_fused_d2q9(int, bool, const FusedItem *, int, const FusedSim *, int,
                             hipStream_t s) {
    run("fused", s);
    return hipSuccess;
}
hipError_t launch_fused_block(int, bool, const FusedTable &t, int, hipStream_t s) {
    last_rows = t.rows;
    run("fused block", s);
    return hipSuccess;
}
int fused_ws_max_comp() { return 10; }
bool fused_ws_fits(int, bool) { return true; }
int fused_ws_blocks_per_cu(int, bool) { return 1; }
hipError_t launch_fused_d2q9_ws(int, bool, const FusedItem *, int, const FusedSim *, int,
                                hipStream_t s) {
    run("fused ws", s);
    return hipSuccess;
}
int field_max_comp() { return 10; }
int field_single_comp() { return 3; }
int field_blocks_per_cu2d(int, bool) { return 1; }
hipError_t launch_field_moments2d(const FieldRun &, bool, hipStream_t s) {
    run("field moments", s);
    return hipSuccess;
}
hipError_t launch_field_eos2d(const FieldRun &, int, int, hipStream_t s) {
    run("field eos", s);
    return hipSuccess;
}
hipError_t launch_field_step2d(const FieldRun &q, int, bool, bool last, int, hipStream_t s) {
    last_rows = q.rows;
    last_members = q.nm;
    run(last ? "field last" : (q.single ? "field single" : "field step"), s);
    return hipSuccess;
}
// FP64 at two wavefronts a SIMD, FP32 storage at three
int field3_blocks_per_cu(bool fp32, int waves) { return (fp32 ? 12 : 8) / waves; }
hipError_t launch_field_moments3(const FieldRun3 &, bool, hipStream_t s) {
    run("field3 moments", s);
    return hipSuccess;
}
hipError_t launch_field_step3(const FieldRun3 &q, int, bool, int, hipStream_t s) {
    stream3_items = q.nitems;
    stream3_waves = q.waves;
    stream3_tiles = q.tiles;
    run("field3 step", s);
    return hipSuccess;
}
hipError_t launch_field_last3(const FieldRun3 &, bool, int, hipStream_t s) {
    run("field3 last", s);
    return hipSuccess;
}

// ---- simulations -------------------------------------------------------------
static fuglbm_mixture *mixture(int n, double tau = 1.0) {
    std::vector<double> Tc, pc, w, M;
    for (int i = 0; i < n; ++i) {
        Tc.push_back(190.6 + 45.0 * i);
        pc.push_back(45.99 - 2.4 * i);
        w.push_back(0.011 + 0.05 * i);
        M.push_back(16.043 + 14.027 * i);
    }
    fuglbm_mixture_desc d;
    std::memset(&d, 0, sizeof(d));
    d.ncomp = n;
    d.Tc_K = Tc.data();
    d.pc_bar = pc.data();
    d.omega = w.data();
    d.M_gmol = M.data();
    d.T_K = 325.0;
    d.kappa_ref_lu = 0.02;
    d.tau = tau;
    fuglbm_mixture *m = nullptr;
    if (fuglbm_init_mixture(&d, &m) != FUGLBM_OK) fault("init_mixture");
    return m;
}

struct Sim {
    fuglbm_mixture *m;
    fuglbm_sim *s = nullptr;
    Sim(int n, int nx, int ny, int nz = 0, double tau = 1.0,
        fuglbm_precision prec = FUGLBM_FP64) {
        m = mixture(n, tau);
        const size_t ns = (size_t)nx * ny * (nz ? nz : 1);
        std::vector<double> rho(ns * n, 0.01);
        if (fuglbm_init_fields(m, nz ? FUGLBM_D3Q19 : FUGLBM_D2Q9, prec, nx, ny, nz ? nz : 1,
                               rho.data(), nullptr, nullptr, &s) != FUGLBM_OK)
            fault(std::string("init_fields: ") + fuglbm_last_error());
    }
    Sim(const Sim &) = delete;
    ~Sim() {
        fuglbm_destroy_sim(s);
        fuglbm_destroy_mixture(m);
    }
    void step(int64_t n) {
        if (fuglbm_step_n(s, n, nullptr) != FUGLBM_OK) fault(fuglbm_last_error());
    }
};
static void step_many(std::vector<Sim *> v, int64_t n) {
    std::vector<fuglbm_sim *> h;
    for (auto *s : v) h.push_back(s->s);
    if (fuglbm_step_many(h.data(), (int32_t)h.size(), n, nullptr) != FUGLBM_OK)
        fault(fuglbm_last_error());
}
static int form_of(const Sim &s) {
    int32_t f = -1;
    if (fuglbm_get_form(s.s, &f) != FUGLBM_OK) fault("get_form");
    return f;
}

static int took(const std::string &kernel) {
    const int n = launched[kernel];
    launched[kernel] = 0;
    return n;
}
// Times of a launch (ms): D2Q9 steps on the fused kernels and in field form,
// and the field form's read of the populations.
static void times(double fused, double step, double moments) {
    cost["fused"] = cost["fused ws"] = cost["fused block"] = fused;
    cost["field step"] = cost["field single"] = step;
    cost["field eos"] = 0.0;
    cost["field moments"] = moments;
}

// ---- scenarios -----------------------------------------------------------------

// A run in field form followed at once by one that does not pay in it: the
// field form's graph may still run and stays.
static void graph_in_flight() {
    times(1.0, 0.9, 10.0);       // pays from 200 steps on
    Sim a(3, 64, 64);
    a.step(1);
    a.step(400);
    CHECK(took("field last") == 1);
    const int before = captures;
    a.step(100);
    CHECK(took("field last") == 0);
    a.step(400);
    CHECK(took("field last") == 1);
    CHECK(captures == before + 1);           // that of the fused steps only
    a.step(100);
    CHECK(captures == before + 1);
}

// A batch's plan follows set_tuning of its members.
static void tuning_between_batches() {
    times(1.0, 0.2, 0.1);
    Sim a(3, 64, 64), b(3, 70, 40);
    step_many({&a, &b}, 8);
    CHECK(took("field last") == 1);
    for (Sim *s : {&a, &b}) CHECK(fuglbm_set_tuning(s->s, 2, 2) == FUGLBM_OK);
    launched.clear();
    step_many({&a, &b}, 8);
    CHECK(took("field last") == 0);
    CHECK(took("fused block") == 8 && last_rows == 2);
    for (Sim *s : {&a, &b}) CHECK(fuglbm_set_tuning(s->s, 0, 0) == FUGLBM_OK);
    step_many({&a, &b}, 8);
    CHECK(took("field last") == 1);
    // one member fixed
    CHECK(fuglbm_set_tuning(b.s, 3, 5) == FUGLBM_OK);
    step_many({&a, &b}, 8);
    CHECK(form_of(b) == FUGLBM_FORM_POPULATIONS);
}

// A call of no steps launches nothing and leaves the next one as it would be
// without it.
static void no_steps_first() {
    times(1.0, 0.2, 0.1);
    Sim a(3, 64, 64), b(3, 70, 40), c(2, 9, 8, 7);
    launched.clear();
    step_many({&a, &b, &c}, 0);
    CHECK(launched.empty());
    step_many({&a, &b, &c}, 8);
    CHECK(took("field last") == 1);
}

// The form a run took is reported, a fixed one is taken, and fixed kernels
// keep populations.
static void form_reported_and_fixed() {
    times(1.0, 0.2, 0.1);
    Sim a(3, 64, 64), b(3, 70, 40), c(2, 24, 24, 24), d(2, 64, 64, 0, 0.8), e(4, 64, 64);
    CHECK(form_of(a) == FUGLBM_FORM_AUTO);
    a.step(0);
    CHECK(form_of(a) == FUGLBM_FORM_AUTO);
    a.step(8);
    CHECK(form_of(a) == FUGLBM_FORM_FIELDS);
    a.step(1);
    CHECK(form_of(a) == FUGLBM_FORM_FIELDS || form_of(a) == FUGLBM_FORM_POPULATIONS);
    CHECK(fuglbm_set_tuning(a.s, 2, 4) == FUGLBM_OK);
    a.step(8);
    CHECK(form_of(a) == FUGLBM_FORM_POPULATIONS);
    // fixed: rows of set_tuning, no trials
    CHECK(fuglbm_set_tuning(a.s, 0, 7) == FUGLBM_OK);
    for (int f : {FUGLBM_FORM_FIELDS, FUGLBM_FORM_FIELDS_SINGLE}) {
        CHECK(fuglbm_set_form(a.s, f) == FUGLBM_OK);
        CHECK(fuglbm_set_form(b.s, f) == FUGLBM_OK);
        launched.clear();
        a.step(1);
        CHECK(form_of(a) == f && took("field last") == 1 && last_rows == 7);
        CHECK(took("fused") + took("fused ws") + took("fused block") == 0);
        a.step(5);
        CHECK(took(f == FUGLBM_FORM_FIELDS ? "field step" : "field single") == 4);
        step_many({&a, &b}, 3);
        CHECK(form_of(a) == f && form_of(b) == f && took("field last") == 2);
        CHECK(took(f == FUGLBM_FORM_FIELDS ? "field step" : "field single") == 2);
        CHECK(took("fused") + took("fused ws") + took("fused block") == 0);
    }
    CHECK(fuglbm_set_form(a.s, FUGLBM_FORM_POPULATIONS) == FUGLBM_OK);
    a.step(8);
    step_many({&a, &b}, 3);
    CHECK(form_of(a) == FUGLBM_FORM_POPULATIONS && form_of(b) == FUGLBM_FORM_FIELDS_SINGLE);
    // D3Q19: the four passes where a caller asks for them
    c.step(8);
    CHECK(form_of(c) == FUGLBM_FORM_FIELDS && took("field3 last") == 1);
    CHECK(fuglbm_set_tuning(c.s, 1, 0) == FUGLBM_OK);
    c.step(8);
    CHECK(form_of(c) == FUGLBM_FORM_POPULATIONS && took("passes") == 8);
    step_many({&c}, 8);
    CHECK(form_of(c) == FUGLBM_FORM_POPULATIONS && took("passes batch") == 8);
    CHECK(fuglbm_set_tuning(c.s, 0, 0) == FUGLBM_OK);
    c.step(8);
    CHECK(form_of(c) == FUGLBM_FORM_FIELDS);
    CHECK(fuglbm_set_form(c.s, FUGLBM_FORM_FIELDS) == FUGLBM_OK);
    c.step(1);
    CHECK(form_of(c) == FUGLBM_FORM_FIELDS);
    // refused
    CHECK(fuglbm_set_form(c.s, FUGLBM_FORM_FIELDS_SINGLE) == FUGLBM_EINVAL);
    CHECK(fuglbm_set_form(d.s, FUGLBM_FORM_FIELDS) == FUGLBM_EINVAL);
    CHECK(fuglbm_set_form(e.s, FUGLBM_FORM_FIELDS_SINGLE) == FUGLBM_EINVAL);
    CHECK(fuglbm_set_form(e.s, 4) == FUGLBM_EINVAL && fuglbm_set_form(e.s, -1) == FUGLBM_EINVAL);
    CHECK(fuglbm_set_form(nullptr, 0) == FUGLBM_EINVAL);
    CHECK(fuglbm_get_form(e.s, nullptr) == FUGLBM_EINVAL);
}

// The tiles of the D3Q19 stream kernel count what is resident at a time: 48^3 x
// 10 in FP64 takes one round of 512 workgroups of four wavefronts, in FP32
// storage one of 768.
static void tiles_that_are_resident() {
    Sim a(10, 48, 48, 48), b(10, 48, 48, 48, 1.0, FUGLBM_FP32_STORAGE);
    CHECK(fuglbm_set_form(a.s, FUGLBM_FORM_FIELDS) == FUGLBM_OK);
    a.step(3);
    CHECK(stream3_waves == 4 && stream3_tiles.W == 16 && stream3_tiles.zc == 2);
    CHECK(stream3_items == 384);
    CHECK(fuglbm_set_form(b.s, FUGLBM_FORM_FIELDS) == FUGLBM_OK);
    b.step(3);
    CHECK(stream3_waves == 4 && stream3_tiles.W == 16 && stream3_tiles.zc == 1);
    CHECK(stream3_items == 768);
}

// The form of a D3Q19 run follows what either is estimated to take, for small
// grids of several components and narrow ones too.
static void cube_forms_by_estimate() {
    struct {
        int n, nx, ny, nz;
        fuglbm_precision prec;
        bool fields;
    } cases[] = {
        // N, shape, storage: measured passes / fields, us
        {3, 24, 24, 24, FUGLBM_FP64, true},              // 26 / 22
        {3, 8, 96, 96, FUGLBM_FP64, true},               // 70 / 39
        {8, 12, 132, 50, FUGLBM_FP32_STORAGE, true},     // 112 / 64
        {10, 64, 64, 64, FUGLBM_FP64, true},             // 199 / 157
        {2, 9, 8, 7, FUGLBM_FP64, true},                 // 21 / 17
        {10, 32, 17, 96, FUGLBM_FP32_STORAGE, false},    // 69 / 84
        {10, 48, 48, 48, FUGLBM_FP32_STORAGE, false},    // 85 / 93
        {10, 27, 10, 9, FUGLBM_FP64, false},             // 48 / 55
    };
    for (auto &k : cases) {
        Sim s(k.n, k.nx, k.ny, k.nz, 1.0, k.prec);
        s.step(2);
        CHECK(form_of(s) == FUGLBM_FORM_POPULATIONS);
        s.step(3);
        if ((form_of(s) == FUGLBM_FORM_FIELDS) != k.fields)
            fault("form of " + std::to_string(k.n) + " x " + std::to_string(k.nx) + " " +
                  std::to_string(k.ny) + " " + std::to_string(k.nz));
    }
}

// A D3Q19 member takes the form it would take, whatever else is in the batch:
// a small one does not send a large one back to the passes.
static void cubes_routed_one_by_one() {
    Sim big(10, 80, 80, 80), small(10, 24, 24, 24), tiny(10, 27, 10, 9), old(3, 20, 20, 20, 0.8),
        fixed(10, 27, 10, 9);
    CHECK(fuglbm_set_form(fixed.s, FUGLBM_FORM_FIELDS) == FUGLBM_OK);
    launched.clear();
    step_many({&small, &big, &tiny, &old}, 5);
    CHECK(form_of(big) == FUGLBM_FORM_FIELDS && took("field3 last") == 1);
    CHECK(form_of(small) == FUGLBM_FORM_POPULATIONS && form_of(tiny) == FUGLBM_FORM_POPULATIONS);
    CHECK(form_of(old) == FUGLBM_FORM_POPULATIONS);
    CHECK(took("passes batch") == 10);          // tau = 1 and tau = 0.8, five steps each
    step_many({&small, &big, &tiny}, 1);        // all share the passes
    CHECK(last_members == 3 && took("passes batch") == 1 && took("field3 last") == 0);
    step_many({&small, &big, &tiny}, 5);
    CHECK(last_members == 2 && took("passes batch") == 5 && took("field3 last") == 1);
    step_many({&tiny, &fixed}, 2);
    CHECK(form_of(fixed) == FUGLBM_FORM_FIELDS && form_of(tiny) == FUGLBM_FORM_POPULATIONS);
    // two that would take it alone share the passes' launches instead, where
    // those cost less than what each adds to them
    Sim a(6, 24, 24, 24), b(6, 24, 24, 24), c(6, 24, 24, 24);
    a.step(5);
    CHECK(form_of(a) == FUGLBM_FORM_FIELDS);
    step_many({&a, &b, &c}, 5);
    CHECK(form_of(a) == FUGLBM_FORM_POPULATIONS && form_of(c) == FUGLBM_FORM_POPULATIONS);
}

static int field_launches() {
    return took("field moments") + took("field eos") + took("field step") + took("field single") +
           took("field last");
}

// Calls of single steps do not time a form that they cannot take; the first
// longer run does, once per shape.
static void single_steps_time_no_field_form() {
    times(1.0, 0.2, 0.1);
    Sim a(3, 64, 64), b(3, 64, 64), c(4, 70, 40), d(4, 50, 30);
    for (int k = 0; k < 3; ++k) {
        a.step(1);
        step_many({&c, &d}, 1);
    }
    CHECK(field_launches() == 0);
    a.step(8);
    CHECK(form_of(a) >= FUGLBM_FORM_FIELDS);
    const int first = field_launches();
    b.step(1);
    b.step(8);
    CHECK(form_of(b) == form_of(a));
    CHECK(field_launches() == 1 + 8 + 8 && first > 17);
    step_many({&c, &d}, 8);
    CHECK(form_of(c) == FUGLBM_FORM_FIELDS);
    CHECK(field_launches() > 17);
    step_many({&c, &d}, 8);
    CHECK(field_launches() == 17);
    step_many({&c, &d}, 1);
    CHECK(form_of(c) == FUGLBM_FORM_POPULATIONS && field_launches() == 0);
}

// D2Q9 members that have a field form take it beside members that do not
// (tau = 0.8, fixed rows), where it saves more than the launches of the
// others; and all share a table where it does not.
static void planes_routed_by_form() {
    times(1.0, 0.2, 0.1);
    Sim a(3, 64, 64), b(3, 70, 40), c(3, 50, 30, 0, 0.8), d(3, 60, 60);
    CHECK(fuglbm_set_tuning(d.s, 2, 2) == FUGLBM_OK);
    step_many({&a, &c, &b, &d}, 8);
    launched.clear();
    step_many({&a, &c, &b, &d}, 8);
    CHECK(took("field last") == 1 && last_members == 2);
    CHECK(took("fused") + took("fused ws") + took("fused block") == 8);
    for (Sim *s : {&a, &b}) CHECK(form_of(*s) >= FUGLBM_FORM_FIELDS);
    for (Sim *s : {&c, &d}) CHECK(form_of(*s) == FUGLBM_FORM_POPULATIONS);
    step_many({&a, &c, &b, &d}, 1);
    CHECK(took("fused") + took("fused ws") + took("fused block") == 1);
    // saves 5 us a step: not worth a launch more
    times(0.105, 0.100, 0.001);
    Sim e(5, 64, 64), f(5, 50, 30, 0, 0.8);
    step_many({&e, &f}, 8);
    CHECK(form_of(e) == FUGLBM_FORM_POPULATIONS);
    launched.clear();
    step_many({&e, &f}, 8);
    CHECK(took("fused") + took("fused ws") + took("fused block") == 8);
    step_many({&e}, 8);
    CHECK(form_of(e) == FUGLBM_FORM_FIELDS);
}

// Read-outs and checkpoints of a simulation's whole life: what is small, or
// read once, or written, makes no pinned ring; what is large or read again does.
static void staging_made_where_it_pays() {
    for (auto prec : {FUGLBM_FP64, FUGLBM_FP32_STORAGE})
        for (int nz : {0, 5}) {      // the host orders these: there and back
            Sim s(2, 13, 7, nz, 1.0, prec);
            const int Q = nz ? 19 : 9;
            std::vector<double> g((size_t)2 * Q * 13 * 7 * (nz ? nz : 1)), h(g.size());
            for (size_t k = 0; k < g.size(); ++k) g[k] = 1.0 / (double)(k + 3);
            launched.clear();
            CHECK(fuglbm_write_populations(s.s, g.data(), 0) == FUGLBM_OK);
            CHECK(fuglbm_read_populations(s.s, h.data()) == FUGLBM_OK);
            CHECK(launched.empty());
            const size_t plane = g.size() / (2 * Q);
            bool equal = true;
            for (size_t k = 0; k < g.size(); ++k)
                equal = equal && h[k] == (prec == FUGLBM_FP64 || k / plane % Q == 0
                                              ? g[k] : (double)(float)g[k]);
            CHECK(equal);
        }
    CHECK(pinned_calls == 0);
    for (int k = 0; k < 3; ++k) {    // 0.9 MB, once each in a life
        Sim s(3, 64, 64);
        std::vector<double> g((size_t)27 * 4096, 0.01);
        CHECK(fuglbm_write_populations(s.s, g.data(), 0) == FUGLBM_OK);
        CHECK(fuglbm_read_populations(s.s, g.data()) == FUGLBM_OK);
    }
    CHECK(pinned_calls == 0);
    {
        Sim s(3, 256, 256);          // 14 MB written, then read
        std::vector<double> g((size_t)27 * 65536, 0.01);
        CHECK(fuglbm_write_populations(s.s, g.data(), 0) == FUGLBM_OK);
        CHECK(pinned_calls == 0);
        CHECK(fuglbm_read_populations(s.s, g.data()) == FUGLBM_OK);
        CHECK(pinned_calls == 1 && pinned_bytes == (size_t)32 << 20);
        CHECK(fuglbm_read_populations(s.s, g.data()) == FUGLBM_OK);
        CHECK(pinned_calls == 1);
    }
    {
        Sim s(3, 90, 90);            // 1.7 MB: from the third time on
        std::vector<double> g((size_t)27 * 8100);
        for (int k = 0; k < 2; ++k) CHECK(fuglbm_read_populations(s.s, g.data()) == FUGLBM_OK);
        CHECK(pinned_calls == 1);
        for (int k = 0; k < 2; ++k) CHECK(fuglbm_read_populations(s.s, g.data()) == FUGLBM_OK);
        CHECK(pinned_calls == 2);
    }
}

int main(int argc, char **argv) {
    const std::map<std::string, std::function<void()>> all = {
        {"graph_in_flight", graph_in_flight},
        {"tuning_between_batches", tuning_between_batches},
        {"no_steps_first", no_steps_first},
        {"tiles_that_are_resident", tiles_that_are_resident},
        {"cube_forms_by_estimate", cube_forms_by_estimate},
        {"cubes_routed_one_by_one", cubes_routed_one_by_one},
        {"single_steps_time_no_field_form", single_steps_time_no_field_form},
        {"planes_routed_by_form", planes_routed_by_form},
        {"staging_made_where_it_pays", staging_made_where_it_pays},
        {"form_reported_and_fixed", form_reported_and_fixed},
    };
    if (argc < 2) {
        for (auto &k : all) std::printf("%s\n", k.first.c_str());
        return 0;
    }
    all.at(argv[1])();
    std::printf("%s\n", failures ? "FAILED" : "OK");
    return failures ? 1 : 0;
}
