// Host side of the C ABI declared in include/fuglbm.h: lattice-unit
// constants, buffer carving, launch tables, hipGraph replay, sticky errors.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstring>
#include <functional>
#include <list>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "../../include/fuglbm.h"
#include "kernels.h"

// A roctx range over one library call (visible with rocprofv3
// --marker-trace beside the kernels the call launches).
struct TraceRange {
    explicit TraceRange(const char *name) { roctxRangePushA(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};

namespace {

thread_local std::string g_err;

fuglbm_status fail(fuglbm_status s, const std::string &msg) {
    g_err = msg;
    return s;
}

fuglbm_status hip_fail(hipError_t e, const char *what) {
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return FUGLBM_EDEVICE;
}

#define HIP_TRY(call)                                   \
    do {                                                \
        hipError_t e_ = (call);                         \
        if (e_ != hipSuccess) return hip_fail(e_, #call); \
    } while (0)

// Cubic equations of state p = RT/(v - b) - a alpha/((v + d1 b)(v + d2 b)):
// a = omega_a R^2 Tc^2 / pc, b = omega_b R Tc / pc put the critical point at
// (Tc, pc); u = d1 + d2 and w = d1 d2 are kept exact.
struct CubicEos {
    double omega_a, omega_b, d1, d2, u, w;
};

CubicEos cubic_eos(int eos) {
    const double s2 = std::sqrt(2.0);
    const double c2 = std::pow(2.0, 1.0 / 3.0);
    switch (eos) {
        case FUGLBM_EOS_SRK:   // Soave-Redlich-Kwong
            return {1.0 / (9.0 * (c2 - 1.0)), (c2 - 1.0) / 3.0, 1.0, 0.0, 1.0, 0.0};
        case FUGLBM_EOS_VDW:   // van der Waals
            return {27.0 / 64.0, 1.0 / 8.0, 0.0, 0.0, 0.0, 0.0};
        default:               // Peng-Robinson, the paper's (Section II.C)
            return {0.457235529, 0.077796074, 1.0 + s2, 1.0 - s2, 2.0, -1.0};
    }
}

// alpha_i(T): PR as in Section II.C (two branches split at omega = 0.49);
// SRK with Soave's m(omega); 1 for vdW.
double cubic_alpha(int eos, double w, double Tr) {
    if (eos == FUGLBM_EOS_VDW) return 1.0;
    double m;
    if (eos == FUGLBM_EOS_SRK)
        m = 0.480 + 1.574 * w - 0.176 * w * w;
    else
        m = w <= 0.49 ? 0.374640 + 1.54226 * w - 0.26992 * w * w
                      : 0.379642 + 1.48503 * w - 0.164423 * w * w + 0.016666 * w * w * w;
    const double sa = 1.0 + m * (1.0 - std::sqrt(Tr));
    return sa * sa;
}

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

int lattice_Q(int lat) { return lat == 0 ? 9 : 19; }
int lattice_D(int lat) { return lat == 0 ? 2 : 3; }

// Fused-kernel rows per work item.  A work item re-reads 4 warm-up rows, so
// longer items waste less; items run in rounds of (CUs x resident
// workgroups per CU).  Pick rows (>= 8, <= ny) minimising
// rounds * (rows + 4).
int compute_units() {
    static int cus = 0;
    if (!cus) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            v > 0)
            cus = v;
        else
            cus = 256;
    }
    return cus;
}

// Fused variants: 2 = register-ring kernel, 3 = store-wave kernel.
bool ws_usable(int ncomp, bool fp32) {
    return ncomp <= fused_ws_max_comp() && fused_ws_fits(ncomp, fp32) &&
           fused_ws_blocks_per_cu(ncomp, fp32) > 0;
}

int blocks_per_cu(int kernel, int ncomp, bool fp32) {
    return kernel == 3 ? fused_ws_blocks_per_cu(ncomp, fp32) : fused_blocks_per_cu(ncomp, fp32);
}

// Variant 2 takes items of one or two rows with the block kernel (all rows
// of an item at once instead of marching): small grids, where a step is a
// chain of latencies.
hipError_t launch_fused(int kernel, int ncomp, bool fp32, const FusedTable &t, int flip,
                        hipStream_t st) {
    if (kernel == 3)
        return launch_fused_d2q9_ws(ncomp, fp32, t.items, t.nitems, t.sims, flip, st);
    if (t.rows <= FUSED_BLOCK_ROWS && ncomp <= FUSED_BLOCK_COMP)
        return launch_fused_block(ncomp, fp32, t, flip, st);
    return launch_fused_d2q9(ncomp, fp32, t.items, t.nitems, t.sims, flip, st);
}

// The fused variant used before (or without) timing: the store-wave kernel
// where it is built and fits, else the register-ring kernel.
int default_fused(int ncomp, bool fp32) { return ws_usable(ncomp, fp32) ? 3 : 2; }

int auto_rows(int nx, int ny, int ncomp, bool fp32, int kernel = 2) {
    const int strips = (nx + FUSED_OUT - 1) / FUSED_OUT;
    const int64_t slots = (int64_t)compute_units() * blocks_per_cu(kernel, ncomp, fp32);
    if (ny <= 8) return ny;
    int best = 8;
    int64_t best_cost = INT64_MAX;
    for (int rows = 8; rows <= ny; ++rows) {
        const int64_t items = (int64_t)strips * ((ny + rows - 1) / rows);
        const int64_t rounds = (items + slots - 1) / slots;
        const int64_t cost = rounds * (rows + 4);
        if (cost < best_cost) {
            best_cost = cost;
            best = rows;
        }
    }
    return best;
}

}  // namespace

struct fuglbm_mixture {
    int N;
    int eos;
    double RT;
    double b[FUG_MAXC], aa[FUG_MAXC], sqk[FUG_MAXC], M[FUG_MAXC];
    double aij[FUG_MAXC * FUG_MAXC];
    double tau;
};

// Layout of one simulation's device memory (offsets from base, 256-aligned).
struct Carve {
    size_t buf0, buf1, cst, status, rho, psi, s, j, u, snap, part, fsim, items, total;
    int max_items;
};

static Carve carve(int N, int lat, bool fp32, int nx, int ny, int nz) {
    Carve c{};
    const int64_t ns = (int64_t)nx * ny * nz;
    const int Q = lattice_Q(lat), D = lattice_D(lat);
    const size_t pop = align256((size_t)(fp32 ? PopLayout<float>(N, Q, nx, (int64_t)ny * nz).bytes((int64_t)ny * nz)
                                              : PopLayout<double>(N, Q, nx, (int64_t)ny * nz).bytes((int64_t)ny * nz)));
    size_t o = 0;
    c.buf0 = o; o += pop;
    c.buf1 = o; o += pop;
    c.cst = o; o += align256(sizeof(SimConst));
    c.status = o; o += 256;
    c.rho = o; o += align256((size_t)N * ns * 8);
    c.psi = o; o += align256((size_t)N * ns * 8);
    c.s = o; o += align256((size_t)ns * 8);
    c.j = o; o += align256((size_t)D * ns * 8);
    c.u = o; o += align256((size_t)D * ns * 8);
    c.snap = o; o += align256((size_t)N * ns * 8);
    c.part = o; o += align256(((size_t)1024 + 1) * (N + 1) * DIAG_QUANT * 8);
    c.fsim = o; o += align256(sizeof(FusedSim));
    c.max_items = 0;
    if (lat == 0) {
        const int strips = (nx + FUSED_OUT - 1) / FUSED_OUT;
        c.max_items = strips * ny + 8;   // rows >= 1 per item
    }
    c.items = o; o += align256((size_t)c.max_items * sizeof(FusedItem));
    c.total = o;
    return c;
}

struct GraphCache {
    hipGraphExec_t exec = nullptr;
    int steps = 0;
    int kernel = 0;
    int rows = 0;
};

// Tiles of the D3Q19 stream kernel (field3_shape); W 0: not chosen yet.
struct Shape3 {
    static constexpr double NONE = 1e300;   // cost where no launch can hold the tiles
    int W = 0, waves = 0, zc = 0;
    double cost = 0.0;
    double rounds = 0.0, simd = 0.0;        // wavefronts that share a SIMD
};
// What a step of a D3Q19 simulation takes in four passes and in field form (us).
struct Step3 {
    double passes = 0.0, fields = 0.0;
};
// What the autotuner chose for a shape: the fused variant and its rows per
// item, the field-form rows (0: not timed), and what a step of each
// and the field form's read of the populations took (ms).  fixed: the form is
// the caller's (fuglbm_set_form), nothing was timed.
struct Tuned {
    int kernel = 0, rows = 0, frows = 0;
    bool single = false, fixed = false;
    float fused_ms = 0.f, field_ms = 0.f, moments_ms = 0.f;
};

namespace {
struct Stage;
}

struct fuglbm_sim {
    const fuglbm_mixture *mix;
    int lattice;
    bool fp32;
    int nx, ny, nz, N, Q, D;
    int64_t ns;
    char *base;
    bool owned;
    Carve cv;
    void *buf[2];
    int parity;            // buffer holding the current state
    SimConst hc;           // host copy of the constant block
    SimConst *dc;
    uint32_t *status;
    double *rho_f, *psi_f, *s_f, *j_f, *u_f, *snap, *part;
    FusedSim *fsim;
    FusedItem *items;
    int nitems;
    int kernel;            // 1 generic, 2 fused (register ring), 3 fused (store waves)
    int rows;
    bool auto_kernel;      // fused variant chosen by timing (not fixed by the caller)
    bool autotune;         // rows chosen by timing (not fixed by the caller)
    bool tuned;            // autotune done (or answered from the cache)
    int64_t step;
    int64_t snap_step;
    bool have_snap;
    uint32_t sticky;
    hipStream_t last_stream;
    // recorded on last_stream after each enqueuing call: a call on another
    // stream waits for it on the device (done_valid: the record is current)
    hipEvent_t done;
    bool done_valid;
    GraphCache graph;
    Tuned tune;            // valid with `tuned`
    int form;              // fuglbm_form asked for
    int form_rows;         // FIELDS, FIELDS_SINGLE on D2Q9: rows per item
    int taken;             // fuglbm_form of the last run
    Shape3 shape3;
    hipGraphExec_t fgraph[2];   // field form, by the parity it was captured at
    Stage *stage;          // pinned staging of its device
    // never reused, and renewed when a caller sets the tuning or the form: batch
    // tables key on it, not on the address
    uint64_t uid;
};

// Work about to be enqueued on st waits (on the device) for the
// simulation's earlier work on another stream: its own event, so no
// reference to that stream is kept.
static fuglbm_status order_after(fuglbm_sim *s, hipStream_t st) {
    if (s->done_valid && s->last_stream != st) HIP_TRY(hipStreamWaitEvent(st, s->done, 0));
    s->last_stream = st;
    return FUGLBM_OK;
}

static fuglbm_status mark_done(fuglbm_sim *s, hipStream_t st) {
    HIP_TRY(hipEventRecord(s->done, st));
    s->done_valid = true;
    s->last_stream = st;
    return FUGLBM_OK;
}

static int64_t pop_bytes(const fuglbm_sim *s) {
    const int64_t rows = (int64_t)s->ny * s->nz;
    return s->fp32 ? PopLayout<float>(s->N, s->Q, s->nx, rows).bytes(rows)
                   : PopLayout<double>(s->N, s->Q, s->nx, rows).bytes(rows);
}

// The fused kernel indexes a buffer with 32-bit element offsets.
static bool fused_fits(const fuglbm_sim *s) {
    const int64_t elems = pop_bytes(s) / (s->fp32 ? 4 : 8);
    return s->lattice == FUGLBM_D2Q9 && elems < ((int64_t)1 << 32);
}

// Launch variants: 1 = four-pass generic kernels, 2 / 3 = fused one-pass
// D2Q9 kernels (register ring / store wavefronts).
static bool is_fused(int kernel) { return kernel == 2 || kernel == 3; }

// The variant a simulation starts with (and kernel 0 of set_tuning picks).
static int default_kernel(const fuglbm_sim *s) {
    return fused_fits(s) ? default_fused(s->N, s->fp32) : 1;
}

static FusedSim fused_sim(const fuglbm_sim *s) {
    return {s->dc, {s->buf[0], s->buf[1]}, s->status, s->parity, s->nx, s->ny, 0};
}

// Steps in field form (fields2d.h): D2Q9 on the fused kernels, at tau = 1.
static bool field_fits(const fuglbm_sim *s) {
    return is_fused(s->kernel) && s->hc.omega == 1.0 && s->N <= field_max_comp();
}

// The same, with form, variant and rows left to the library.
static bool field_usable(const fuglbm_sim *s) {
    return field_fits(s) && s->form == FUGLBM_FORM_AUTO && s->auto_kernel && s->autotune;
}

// The caller asked for the field form.
static bool form_fixed(const fuglbm_sim *s) { return s->form >= FUGLBM_FORM_FIELDS; }

// Whether a run of n steps is taken in field form.  Beside its steps it
// reads the populations at its start and writes them at its end (about as
// long); both forms give bitwise the same state.  One step never gains.
// step_ms: what every step costs beside it.
static bool field_pays(const Tuned &t, int64_t n, double step_ms = 0.0) {
    if (t.fixed) return true;
    return t.frows > 0 && n >= 2 &&
           (double)n * (t.fused_ms - t.field_ms - step_ms) > 2.0 * t.moments_ms;
}

// All fields lie in the spare population buffer where they fit, components
// a padded stride apart (see PopLayout<float>::pad for the gap): they take 3 N +
// 7 values of a site, the buffer has room for 9 N in FP64 (from two components
// on) and 5 N in FP32 storage (from four on), less the gaps on small grids.
// Else set 0 and psi use the workspace.
static FieldSim field_sim(const fuglbm_sim *s) {
    FieldSim f{};
    f.c = s->dc;
    f.buf[0] = s->buf[0];
    f.buf[1] = s->buf[1];
    f.rho = s->rho_f;
    f.psi = s->psi_f;
    f.s = s->s_f;
    f.j = s->j_f;
    f.u = s->u_f;
    f.status = s->status;
    f.ld = s->ns + PopLayout<float>::pad(s->ns);
    f.wide = (3 * s->N + 3 + 2 * s->D) * f.ld * 8 <= pop_bytes(s);
    if (!f.wide) f.ld = s->ns;
    f.parity = s->parity;
    f.nx = s->nx;
    f.ny = s->ny;
    return f;
}

static FieldRun field_run(const fuglbm_sim *s, int rows, bool single) {
    FieldRun q{};
    q.one = field_sim(s);
    q.strips = (s->nx + FUSED_OUT - 1) / FUSED_OUT;
    q.rows = rows;
    q.nitems = q.strips * ((s->ny + rows - 1) / rows);
    q.blocks = (s->ns + 255) / 256;
    q.single = single;
    return q;
}

// D3Q19 steps in field form (fields3d.h): tau = 1, planes within 32-bit byte
// offsets.
static bool field3_fits(const fuglbm_sim *s) {
    return s->lattice == FUGLBM_D3Q19 && s->kernel == 1 && s->hc.omega == 1.0 && s->N <= field_max_comp() &&
           (int64_t)s->nx * s->ny < ((int64_t)1 << 29) && s->ns < ((int64_t)1 << 31);
}

// The fields of set `set` of a run that reads buf[parity]: all in the spare
// population buffer where they fit (else set 0, psi and u in the workspace).
static GenMember field3_member(const fuglbm_sim *s, int parity, int set) {
    GenMember g{};
    g.c = s->dc;
    g.buf[0] = s->buf[0];
    g.buf[1] = s->buf[1];
    g.status = s->status;
    g.parity = parity;
    const int64_t ns = s->ns, N = s->N;
    double *b = (double *)s->buf[parity ^ 1];
    if ((3 * N + 11) * ns * 8 <= pop_bytes(s)) {
        g.rho_f = b + set * N * ns;
        g.psi_f = b + 2 * N * ns;
        b += 3 * N * ns;
        g.u_f = b;
        g.s_f = b + (3 + set) * ns;
        g.j_f = b + (5 + 3 * set) * ns;
    } else {
        g.rho_f = set ? b : s->rho_f;
        g.s_f = set ? b + N * ns : s->s_f;
        g.j_f = set ? b + (N + 1) * ns : s->j_f;
        g.psi_f = s->psi_f;
        g.u_f = s->u_f;
    }
    return g;
}

static uint64_t next_sim_uid() {
    static std::atomic<uint64_t> n{0};
    return ++n;
}

namespace {

hipStream_t capture_stream() {
    static hipStream_t s = nullptr;
    if (!s) {
        if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) s = nullptr;
    }
    return s;
}

// Work items of one simulation for `rows` rows per item, in launch order.
// Logical order: chunk-major (a band of rows across the full width).
// Workgroups are handed to the 8 XCDs round-robin; XCD k gets the k-th
// contiguous slice of the logical order, so neighbouring items (which
// re-read each other's halo) share that XCD's L2.
std::vector<FusedItem> item_list(const fuglbm_sim *s, int rows) {
    const int strips = (s->nx + FUSED_OUT - 1) / FUSED_OUT;
    const int chunks = (s->ny + rows - 1) / rows;
    std::vector<FusedItem> logical;
    for (int c = 0; c < chunks; ++c)
        for (int t = 0; t < strips; ++t)
            logical.push_back({0, t * FUSED_OUT, c * rows, std::min(rows, s->ny - c * rows)});
    const int n = (int)logical.size();
    const int per = (n + 7) / 8;
    std::vector<FusedItem> it((size_t)per * 8, FusedItem{-1, 0, 0, 0});
    for (int b = 0; b < per * 8; ++b) {
        const int k = b % 8, q = b / 8;
        const int li = k * per + q;
        if (li < n) it[b] = logical[li];
    }
    return it;
}

fuglbm_status build_items(fuglbm_sim *s) {
    const std::vector<FusedItem> it = item_list(s, s->rows);
    if ((int)it.size() > s->cv.max_items) return fail(FUGLBM_EINVAL, "too many work items");
    s->nitems = (int)it.size();
    HIP_TRY(hipMemcpy(s->items, it.data(), it.size() * sizeof(FusedItem), hipMemcpyHostToDevice));
    return FUGLBM_OK;
}

// Every graph of the simulation; its work must have ended.
void drop_graphs(fuglbm_sim *s) {
    if (s->graph.exec) (void)hipGraphExecDestroy(s->graph.exec);
    s->graph = GraphCache{};
    for (auto &g : s->fgraph) {
        if (g) (void)hipGraphExecDestroy(g);
        g = nullptr;
    }
}

hipError_t launch_one_step(fuglbm_sim *s, int flip_parity, hipStream_t st) {
    if (is_fused(s->kernel))
        return launch_fused(s->kernel, s->N, s->fp32,
                            {s->items, s->nitems, s->fsim, 1, s->rows}, flip_parity, st);
    return launch_step_generic(s->lattice, s->fp32, s->dc, s->N, s->nx, s->ny, s->nz, s->buf[flip_parity],
                               s->buf[flip_parity ^ 1], s->rho_f, s->psi_f, s->s_f, s->j_f,
                               s->u_f, s->status, s->hc.omega != 1.0, st);
}

constexpr int GRAPH_STEPS = 32;  // even: a replay returns to the same parity

// Captures GRAPH_STEPS calls of launch(k, stream) and instantiates the graph.
template <class Launch>
fuglbm_status capture_steps(Launch launch, hipGraphExec_t &ex, const char *what) {
    hipStream_t cs = capture_stream();
    if (!cs) return fail(FUGLBM_EDEVICE, "cannot create capture stream");
    HIP_TRY(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    for (int k = 0; k < GRAPH_STEPS; ++k) {
        hipError_t e = launch(k, cs);
        if (e != hipSuccess) {
            hipGraph_t g = nullptr;
            if (hipStreamEndCapture(cs, &g) == hipSuccess && g) (void)hipGraphDestroy(g);
            return hip_fail(e, what);
        }
    }
    hipGraph_t g = nullptr;
    HIP_TRY(hipStreamEndCapture(cs, &g));
    hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        ex = nullptr;
        return hip_fail(e, what);
    }
    return FUGLBM_OK;
}

fuglbm_status ensure_graph(fuglbm_sim *s) {
    if (s->graph.exec && s->graph.kernel == s->kernel && s->graph.rows == s->rows)
        return FUGLBM_OK;
    // only this form's graph: one of the field form may be running, and stays
    // valid
    if (s->graph.exec) {
        HIP_TRY(hipStreamSynchronize(s->last_stream));
        (void)hipGraphExecDestroy(s->graph.exec);
        s->graph = GraphCache{};
    }
    fuglbm_status rc = capture_steps(
        [&](int k, hipStream_t cs) { return launch_one_step(s, k & 1, cs); }, s->graph.exec,
        "step graph");
    if (rc != FUGLBM_OK) return rc;
    s->graph.steps = GRAPH_STEPS;
    s->graph.kernel = s->kernel;
    s->graph.rows = s->rows;
    return FUGLBM_OK;
}

// One step in field form from set `set` (last: to the populations).
hipError_t launch_field(const FieldRun &q, int ncomp, bool fp32, bool last, int set,
                        hipStream_t st) {
    hipError_t e = launch_field_eos2d(q, ncomp, set, st);
    return e != hipSuccess ? e : launch_field_step2d(q, ncomp, fp32, last, set, st);
}

bool capturing(hipStream_t st) {
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &c) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return c != hipStreamCaptureStatusNone;
}

// n >= 1 steps in field form: first() makes set 0 from the populations,
// step(set, stream) takes a set to the other one, last(set) to the
// populations.  They end in the buffer they started from (the other one held
// the fields), so no parity changes.  graph: a captured run of GRAPH_STEPS
// steps (set 0 to set 0), made when it is first needed; a caller that
// captures the stream gets plain launches up to the run length at which the
// steps of the other forms come from a graph.
template <class First, class Step, class Last>
fuglbm_status field_steps(First first, Step step, Last last, int64_t n, hipGraphExec_t &graph,
                          hipStream_t st) {
    HIP_TRY(first());
    int64_t left = n - 1;
    if (left >= 2 * GRAPH_STEPS || (graph && left >= GRAPH_STEPS && !capturing(st))) {
        if (!graph) {
            fuglbm_status rc = capture_steps([&](int k, hipStream_t cs) { return step(k & 1, cs); },
                                             graph, "field step graph");
            if (rc != FUGLBM_OK) return rc;
        }
        for (; left >= GRAPH_STEPS; left -= GRAPH_STEPS) HIP_TRY(hipGraphLaunch(graph, st));
    }
    int set = 0;
    for (; left > 0; --left, set ^= 1) HIP_TRY(step(set, st));
    HIP_TRY(last(set));
    return FUGLBM_OK;
}

fuglbm_status run_field(const FieldRun &q, int ncomp, bool fp32, int64_t n, hipGraphExec_t &graph,
                        hipStream_t st) {
    return field_steps([&] { return launch_field_moments2d(q, fp32, st); },
                       [&](int set, hipStream_t to) {
                           return launch_field(q, ncomp, fp32, false, set, to);
                       },
                       [&](int set) { return launch_field(q, ncomp, fp32, true, set, st); }, n,
                       graph, st);
}

// ---- D3Q19 in field form --------------------------------------------------
// Tiles of the stream kernel.  A workgroup collides W x R sites a plane for
// (W - 4) x (R - 2) of output, and its two rim planes cost 0.9 of a plane,
// so wide, tall and long tiles waste least; but all of them should be
// resident at once (as many to a CU as the kernel's registers allow: 8
// wavefronts in FP64, 12 in FP32 storage), and a SIMD works through its
// wavefronts one after another.  The cheapest of the widths, heights and chunk lengths by
//   cost = rounds x (zc + 0.9) x wavefronts per SIMD (at least 2: latency)
//          x components,
// planes of one wavefront that a SIMD works through.
const Shape3 &field3_shape(fuglbm_sim *s) {
    if (s->shape3.W) return s->shape3;
    const int most = s->fp32 ? 12 : 8, cus = compute_units();
    Shape3 best{32, most, 1, Shape3::NONE};
    for (int waves = 4; waves <= most; waves += 4) {
        const int per_cu = field3_blocks_per_cu(s->fp32, waves), slots = cus * per_cu;
        for (int W = 16; W <= 64; W *= 2) {
            const int R = 64 * waves / W;
            const int64_t cols = (int64_t)((s->nx + W - 5) / (W - 4)) * ((s->ny + R - 3) / (R - 2));
            // chunk lengths: the shortest for each count of chunks
            for (int zc = 1, tz = 0; tz != 1; zc = tz > 1 ? (s->nz + tz - 2) / (tz - 1) : zc) {
                tz = (s->nz + zc - 1) / zc;
                const int64_t items = cols * tz;
                if ((items + 7) * 64 * waves >= (int64_t)1 << 32) continue;   // threads of a launch
                const double rounds = (double)((items + slots - 1) / slots);
                const int resident = (int)std::min<int64_t>(per_cu, (items + cus - 1) / cus);
                const double per_simd = std::max(2.0, waves * resident / 4.0);
                const double cost = rounds * (zc + 0.9) * per_simd * s->N;
                if (cost < best.cost)
                    best = {W, waves, zc, cost, rounds, waves * resident / 4.0};
            }
        }
    }
    return s->shape3 = best;
}

// What the four passes take beside their volume (us): launches and latencies,
// which the members of a batch share.
double step3_latency(int ncomp) { return 14.0 + 3.2 * ncomp; }

// What a step takes in either form (us).  The four passes: latencies
// (components one after another); sites and components, more where rows are
// not whole 64-byte lines, so that the collision writes parts of them, and
// more again for those past what the last-level cache holds; and the sites
// that the 64 x 2 x 2 tiles of the collision cover.  The field form: latencies,
// the planes that a SIMD works through (the more wavefronts share it the longer
// each takes), the EOS by sites and components, and the velocity pass by the
// sites that its 16 x 4 x 4 tiles cover.
//
// Fitted to 616 pairs of steps measured in runs of 65 (N = 1 ... 10, 9 7 8 ...
// 128^3, widths from 8, both precisions): 5 and 3 % off (rms).  Over 300 other
// pairs the form they pick is the slower one by 5.7 % at worst (16 57 9, N = 10,
// FP32 storage: passes 52.2, fields 55.2 us) and 0.1 % in the mean; thresholds on
// sites per cost, which these replace, lost up to 83 % (8 96 96, N = 3: 65.7 and
// 36.0 us) and 5 % in the mean.  FP32 storage's estimate of the field form is
// taken 3 % up, where fewer near ties go the wrong way.  Far from a
// tie: 128^3 x 10 FP64 1868 / 973, FP32 storage 1210 / 892; 32 17 96, N = 10,
// FP32 storage 69 / 84.  Trials at the first run of a shape were no better:
// short ones find the clocks low, which the field form's VALU work feels more
// (64^3 x 10 FP64: 203 / 199 in trials of four steps, 199 / 157 in a run).
Step3 step3_estimate(fuglbm_sim *s) {
    const double n = s->N, sites = 1e-6 * (double)s->ns, work = sites * n;
    const bool lines = s->nx % (s->fp32 ? 16 : 8) == 0;
    int64_t units[3];
    generic_units(1, s->N, s->nx, s->ny, s->nz, units);
    const double velocity = 256e-6 * (double)units[1] * n, collision = 256e-6 * (double)units[2];
    const double far = std::max(0.0, work - (s->fp32 ? 0.8 : 0.5));
    const Shape3 &h = field3_shape(s);
    Step3 e;
    e.passes = step3_latency(s->N) + 39.0 * sites + 20.5 * collision;
    e.fields = 22.0 * sites;
    if (s->fp32) {
        e.passes += lines ? 4.0 * work + 21.0 * far : 5.0 * work + 27.0 * far;
        e.fields += 8.1 + 3.7 * n + 7.2 * work + 4.1 * velocity +
                    (1.21 * h.simd - 0.44) * h.rounds * h.zc * n;
    } else {
        e.passes += lines ? 15.0 * work + 24.0 * far : 21.0 * work + 53.0 * far;
        e.fields += 7.9 + 3.9 * n + 8.0 * work + 4.0 * velocity +
                    (1.36 * h.simd - 0.58) * h.rounds * h.zc * n;
    }
    return e;
}

// A run of n steps whose form the library chooses (from three steps on).
bool field3_open(fuglbm_sim *s, int64_t n) {
    return n >= 3 && s->form == FUGLBM_FORM_AUTO && field3_fits(s) &&
           field3_shape(s).cost < Shape3::NONE;
}

// A simulation on its own takes a run of n steps in field form.
bool field3_alone(fuglbm_sim *s, int64_t n) {
    if (!field3_open(s, n)) return form_fixed(s) && field3_fits(s);
    const Step3 c = step3_estimate(s);
    return c.fields < c.passes;
}

// Members of a D3Q19 group that take a run of n steps in field form, the
// others in `rest`: those whose caller fixed it, and those whose step is faster
// so than what it adds to the passes that the group shares; or all, where that
// is faster than shared passes for the few that are left.  What a member adds
// is 1.3 times its volume, as every block of a batch looks its member up: three
// 64^3 x 4 take 267 us a step so (FP64; 273 by this) and 212 in field form,
// four 40^3 x 3 90 us (88) and 153, 128^3 x 10 with 20 11 9 x 10 2090 and 975.
void split_forms3(const std::vector<fuglbm_sim *> &group, int64_t n,
                  std::vector<fuglbm_sim *> &fields, std::vector<fuglbm_sim *> &rest) {
    double shared = 0.0, apart = 0.0, latency = 0.0;
    bool all = true;   // every one in `rest` may take the field form
    for (auto *s : group) {
        const bool open = field3_open(s, n);
        const double lat = step3_latency(s->N);
        const Step3 c = open ? step3_estimate(s) : Step3{};
        const double adds = 1.3 * (c.passes - lat);
        if ((form_fixed(s) && field3_fits(s)) || (open && c.fields < adds)) {
            fields.push_back(s);
            continue;
        }
        rest.push_back(s);
        all = all && open;
        shared += adds;
        apart += c.fields;
        latency = std::max(latency, lat);
    }
    if (all && apart < shared + latency) {
        fields = group;
        rest.clear();
    }
}

FieldRun3 field3_run(fuglbm_sim *s) {
    FieldRun3 q{};
    const Shape3 h = field3_shape(s);
    const int R = 64 * h.waves / h.W;
    q.f[0] = field3_member(s, s->parity, 0);
    q.f[1] = field3_member(s, s->parity, 1);
    q.ns = s->ns;
    q.waves = h.waves;
    q.tiles = {h.W, h.zc, (s->nx + h.W - 5) / (h.W - 4), (s->ny + R - 3) / (R - 2),
               (s->nz + h.zc - 1) / h.zc};
    q.nitems = (q.tiles.tx * q.tiles.ty * q.tiles.tz + 7) / 8 * 8;
    generic_units(1, s->N, s->nx, s->ny, s->nz, q.total);
    return q;
}

fuglbm_status run_field3(fuglbm_sim *s, int64_t n, hipStream_t st) {
    const FieldRun3 q = field3_run(s);
    const fuglbm_status rc = field_steps(
        [&] { return launch_field_moments3(q, s->fp32, st); },
        [&](int set, hipStream_t to) { return launch_field_step3(q, s->N, s->fp32, set, to); },
        [&](int set) { return launch_field_last3(q, s->fp32, set, st); }, n,
        s->fgraph[s->parity], st);
    if (rc == FUGLBM_OK) {
        s->step += n;
        s->taken = FUGLBM_FORM_FIELDS;
    }
    return rc;
}

// ---- rows-per-item autotuner ---------------------------------------------
// Candidates are timed on trial launches that read the current state and
// write the other buffer without swapping them: the state does not move,
// and the next real step overwrites what the trials wrote.  (Every rows
// value gives bitwise the same new state, since each site's arithmetic does
// not depend on which work item computes it.)  The winner is cached per
// (nx, ny, N, precision) for the process, and per batch shape for batched
// launches.
constexpr int TUNE_ROWS[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256};
constexpr int TUNE_LAUNCHES = 4;

std::vector<int> tune_candidates(int ny, int model) {
    std::vector<int> c;
    for (int r : TUNE_ROWS)
        if (r < ny) c.push_back(r);
    c.push_back(ny);
    if (model > 0 && model < ny) c.push_back(model);
    std::sort(c.begin(), c.end());
    c.erase(std::unique(c.begin(), c.end()), c.end());
    return c;
}

struct Timer {
    hipEvent_t a = nullptr, b = nullptr;
    Timer() {
        if (hipEventCreate(&a) != hipSuccess) a = nullptr;
        if (hipEventCreate(&b) != hipSuccess) b = nullptr;
    }
    ~Timer() {
        if (a) (void)hipEventDestroy(a);
        if (b) (void)hipEventDestroy(b);
    }
    Timer(const Timer &) = delete;
    Timer &operator=(const Timer &) = delete;
    bool ok() const { return a && b; }
};

// Times `launch` (TUNE_LAUNCHES back-to-back launches) after `prepare(r)`
// for every candidate r; returns the fastest.
template <class Prep, class Launch>
// Candidates are timed in two passes, in order and then in reverse order,
// and ranked by the sum: the GPU's clocks still rise during the first
// hundreds of milliseconds of sustained work, so a single pass would favour
// the candidates timed last.
fuglbm_status time_candidates(const std::vector<int> &cand, hipStream_t st, Prep prepare,
                              Launch launch, int &best, float *best_time = nullptr) {
    Timer tm;
    if (!tm.ok()) return fail(FUGLBM_EDEVICE, "hipEventCreate");
    std::vector<float> sum(cand.size(), 0.f);
    bool warm = false;
    for (int pass = 0; pass < 2; ++pass) {
        for (size_t q = 0; q < cand.size(); ++q) {
            const size_t k = pass == 0 ? q : cand.size() - 1 - q;
            fuglbm_status rc = prepare(cand[k]);
            if (rc != FUGLBM_OK) return rc;
            if (!warm) {   // first launch of the kernel: not timed
                HIP_TRY(launch());
                warm = true;
            }
            HIP_TRY(hipEventRecord(tm.a, st));
            for (int j = 0; j < TUNE_LAUNCHES; ++j) HIP_TRY(launch());
            HIP_TRY(hipEventRecord(tm.b, st));
            HIP_TRY(hipEventSynchronize(tm.b));
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, tm.a, tm.b));
            sum[k] += ms;
        }
    }
    float best_ms = 1e30f;
    best = cand.empty() ? 0 : cand[0];
    for (size_t k = 0; k < cand.size(); ++k)
        if (sum[k] < best_ms) {
            best_ms = sum[k];
            best = cand[k];
        }
    if (best_time) *best_time = best_ms;
    return FUGLBM_OK;
}

std::map<std::tuple<int, int, int, int>, Tuned> &tune_cache() {
    static std::map<std::tuple<int, int, int, int>, Tuned> m;
    return m;
}

// Rows per item of the field form whose rounds over the resident workgroups
// cost least (a workgroup takes rows + 6 lead rows, a single wavefront
// rows + 4), with the items of each simulation counted as they are cut:
// 1024^2, N = 10 on 256 slots takes 74 rows (252 items, one round, 121 us a
// step), where strip rows in total would give 72 (270 items, two rounds, 130).
int field_model_rows(const std::vector<const fuglbm_sim *> &sims, bool single) {
    int ny = 1;
    for (auto *s : sims) ny = std::max(ny, s->ny);
    const int64_t slots = (int64_t)compute_units() * field_blocks_per_cu2d(sims[0]->N, single);
    int best = 1;
    int64_t best_cost = INT64_MAX;
    for (int rows = 1; rows <= ny; ++rows) {
        int64_t items = 0;
        for (auto *s : sims)
            items += (int64_t)((s->nx + FUSED_OUT - 1) / FUSED_OUT) * ((s->ny + rows - 1) / rows);
        const int64_t cost = (items + slots - 1) / slots * (rows + (single ? 4 : 6));
        if (cost < best_cost) {
            best_cost = cost;
            best = rows;
        }
    }
    return best;
}

// Times the field form of simulations of up to ny rows over `set_rows(rows)`
// (which gives the run to launch): its moments and EOS kernels once, its step
// kernel and, for few components, the one by single wavefronts at each rows
// candidate; two passes, ranked by the sum.  The trials read the current
// populations and write the spare buffer and workspace only.
template <class SetRows>
fuglbm_status time_field(const std::vector<const fuglbm_sim *> &sims, hipStream_t st,
                         SetRows set_rows, Tuned &t) {
    const int ncomp = sims[0]->N;
    const bool fp32 = sims[0]->fp32;
    int ny = 1;
    for (auto *s : sims) ny = std::max(ny, s->ny);
    const std::vector<int> cand = tune_candidates(ny, field_model_rows(sims, false));
    FieldRun q;
    fuglbm_status rc = set_rows(cand[0], q);
    if (rc != FUGLBM_OK) return rc;
    Timer tm;
    if (!tm.ok()) return fail(FUGLBM_EDEVICE, "hipEventCreate");
    auto timed = [&](auto launch, float &ms) -> fuglbm_status {
        HIP_TRY(hipEventRecord(tm.a, st));
        for (int j = 0; j < TUNE_LAUNCHES; ++j) HIP_TRY(launch());
        HIP_TRY(hipEventRecord(tm.b, st));
        HIP_TRY(hipEventSynchronize(tm.b));
        HIP_TRY(hipEventElapsedTime(&ms, tm.a, tm.b));
        ms /= TUNE_LAUNCHES;
        return FUGLBM_OK;
    };
    auto moments = [&] { return launch_field_moments2d(q, fp32, st); };
    auto eos = [&] { return launch_field_eos2d(q, ncomp, 0, st); };
    float eos_ms = 0.f;
    HIP_TRY(moments());
    HIP_TRY(eos());
    rc = timed(moments, t.moments_ms);
    if (rc == FUGLBM_OK) rc = timed(eos, eos_ms);
    if (rc != FUGLBM_OK) return rc;
    int best = 0;
    float best_ms = 0.f;
    rc = time_candidates(
        cand, st, [&](int r) { return set_rows(r, q); },
        [&] { return launch_field_step2d(q, ncomp, fp32, false, 0, st); }, best, &best_ms);
    if (rc != FUGLBM_OK) return rc;
    t.frows = best;
    t.field_ms = eos_ms + best_ms / (2 * TUNE_LAUNCHES);
    if (ncomp <= field_single_comp()) {
        rc = time_candidates(
            tune_candidates(ny, field_model_rows(sims, true)), st,
            [&](int r) {
                fuglbm_status e = set_rows(r, q);
                q.single = true;
                return e;
            },
            [&] { return launch_field_step2d(q, ncomp, fp32, false, 0, st); }, best, &best_ms);
        if (rc != FUGLBM_OK) return rc;
        const float ms = eos_ms + best_ms / (2 * TUNE_LAUNCHES);
        // clearly faster alone: at 512^2 x 3 the trials call the two equal and
        // a run does not (22.9 / 23.5 us a step)
        if (ms < 0.95f * t.field_ms) {
            t.frows = best;
            t.field_ms = ms;
            t.single = true;
        }
    }
    return FUGLBM_OK;
}

fuglbm_status set_rows(fuglbm_sim *s, int rows, hipStream_t st) {
    if (rows == s->rows) return FUGLBM_OK;
    HIP_TRY(hipStreamSynchronize(st));   // queued launches still read the item table
    s->rows = rows;
    return build_items(s);
}

// With the variant left to the tuner, both fused variants are timed (each
// at its own rows candidates) and the faster (variant, rows) is kept.
// The choice is cached.  Every candidate's work table
// is uploaded once, before any timing, and the candidates run back to back
// with an event pair each and one synchronisation at the end: the GPU
// stays busy through the whole trial, so the candidates are timed under
// the same sustained load (with a host wait between candidates the clocks
// fall back and the early candidates run slower).
std::tuple<int, int, int, int> tune_key(const fuglbm_sim *s) {
    const bool both = s->auto_kernel && ws_usable(s->N, s->fp32);
    const int tag = (both ? 0 : s->kernel) + (field_usable(s) ? 4 : 0);
    return {s->nx, s->ny, s->N, (s->fp32 ? 1 : 0) + 2 * tag};
}

fuglbm_status autotune_rows(fuglbm_sim *s, hipStream_t st) {
    const TraceRange trace_range("fuglbm autotune rows");
    const bool both = s->auto_kernel && ws_usable(s->N, s->fp32);
    const auto key = tune_key(s);
    auto hit = tune_cache().find(key);
    Tuned &tn = s->tune;
    if (hit != tune_cache().end()) {
        tn = hit->second;
    } else {
        tn = Tuned{};
        struct Cand {
            int kernel, rows;
            size_t off, n;
        };
        std::vector<Cand> cand;
        std::vector<FusedItem> all;
        for (int k : {2, 3}) {
            if (both ? false : k != s->kernel) continue;
            if (k == 3 && !ws_usable(s->N, s->fp32)) continue;
            for (int r : tune_candidates(s->ny, auto_rows(s->nx, s->ny, s->N, s->fp32, k))) {
                const std::vector<FusedItem> it = item_list(s, r);
                cand.push_back({k, r, all.size(), it.size()});
                all.insert(all.end(), it.begin(), it.end());
            }
        }
        // the candidates' tables; freed once the stream has drained (also on
        // an early error return, while trial launches may still read them)
        struct DevTables {
            FusedItem *p = nullptr;
            hipStream_t st;
            ~DevTables() {
                if (p) {
                    (void)hipStreamSynchronize(st);
                    (void)hipFree(p);
                }
            }
        } tables{nullptr, st};
        HIP_TRY(hipMalloc(&tables.p, all.size() * sizeof(FusedItem)));
        FusedItem *dev = tables.p;
        HIP_TRY(hipStreamSynchronize(st));
        HIP_TRY(hipMemcpy(dev, all.data(), all.size() * sizeof(FusedItem), hipMemcpyHostToDevice));
        // two passes, in order and in reverse order, ranked by the sum (see
        // time_candidates), queued back to back with one wait at the end
        std::vector<Timer> tm(2 * cand.size());
        for (auto &t : tm)
            if (!t.ok()) return fail(FUGLBM_EDEVICE, "hipEventCreate");
        // the trial launches read the current state and write the spare
        // buffer (parity unchanged): the state does not move
        auto launch = [&](const Cand &c) {
            return launch_fused(c.kernel, s->N, s->fp32,
                                {dev + c.off, (int)c.n, s->fsim, 1, c.rows}, s->parity, st);
        };
        for (size_t i = 0; i < cand.size(); ++i)   // first launch of each variant: not timed
            if (i == 0 || cand[i].kernel != cand[i - 1].kernel) HIP_TRY(launch(cand[i]));
        const size_t nc = cand.size();
        for (size_t q = 0; q < 2 * nc; ++q) {
            const size_t i = q < nc ? q : 2 * nc - 1 - q;
            HIP_TRY(hipEventRecord(tm[q].a, st));
            for (int j = 0; j < TUNE_LAUNCHES; ++j) HIP_TRY(launch(cand[i]));
            HIP_TRY(hipEventRecord(tm[q].b, st));
        }
        HIP_TRY(hipEventSynchronize(tm.back().b));
        float best_ms = 1e30f;
        for (size_t i = 0; i < nc; ++i) {
            float m1 = 0.f, m2 = 0.f;
            HIP_TRY(hipEventElapsedTime(&m1, tm[i].a, tm[i].b));
            HIP_TRY(hipEventElapsedTime(&m2, tm[2 * nc - 1 - i].a, tm[2 * nc - 1 - i].b));
            const float ms = m1 + m2;
            if (ms < best_ms) {
                best_ms = ms;
                tn.kernel = cand[i].kernel;
                tn.rows = cand[i].rows;
            }
        }
        tn.fused_ms = best_ms / (2 * TUNE_LAUNCHES);
        tune_cache()[key] = tn;
    }
    HIP_TRY(hipStreamSynchronize(st));
    s->kernel = tn.kernel;
    s->tuned = true;
    return set_rows(s, tn.rows, st);
}

// The field form beside it, timed at the first run of several steps: programs
// that take single steps do not pay for it.  Once per shape it costs (fused
// variants / field form, ms): 64^2 x 3 9 / 4, 256^2 x 3 26 / 12, 200^2 x 10
// 50 / 7, 1024^2 x 3 83 / 31, 1024^2 x 10 211 / 27; a batch of 12 grids of
// 64^2 ... 152^2 x 3 23 / 14.
fuglbm_status autotune_field(fuglbm_sim *s, hipStream_t st) {
    const TraceRange trace_range("fuglbm autotune field form");
    Tuned &c = tune_cache()[tune_key(s)];
    if (!c.frows) {
        Tuned tn = s->tune;
        fuglbm_status rc = time_field(
            {s}, st,
            [&](int r, FieldRun &q) {
                q = field_run(s, r, false);
                return FUGLBM_OK;
            },
            tn);
        if (rc != FUGLBM_OK) return rc;
        c = tn;
    }
    s->tune = c;
    return FUGLBM_OK;
}

// ---- side streams of a batch ----------------------------------------------
// The groups of a batch (fuglbm_step_many) do not depend on each other, and
// one of a few small grids leaves most of the chip idle: beside the caller's
// stream they run on LANES - 1 side streams, which wait for what the caller's
// stream holds and which it waits for in turn before the call's work counts
// as done.  Four in all, the hardware queues of a process.  Held while any
// simulation exists; a call that finds them in use by another thread runs
// its groups one after another.
constexpr int LANES = 4;

struct Lanes {
    std::mutex use;             // held by the call that enqueues on them
    hipStream_t st[LANES] = {};   // st[0] unused: the caller's
    hipEvent_t fork = nullptr, join[LANES] = {};

    // with `use` held
    bool ready() {
        if (!fork && hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess)
            fork = nullptr;
        bool ok = fork != nullptr;
        for (int k = 1; k < LANES && ok; ++k) {
            if (!st[k] && hipStreamCreateWithFlags(&st[k], hipStreamNonBlocking) != hipSuccess)
                st[k] = nullptr;
            if (!join[k] && hipEventCreateWithFlags(&join[k], hipEventDisableTiming) != hipSuccess)
                join[k] = nullptr;
            ok = st[k] && join[k];
        }
        if (!ok) (void)hipGetLastError();
        return ok;
    }
    void release() {
        std::lock_guard<std::mutex> g(use);
        for (int k = 1; k < LANES; ++k) {
            if (st[k]) (void)hipStreamDestroy(st[k]);
            if (join[k]) (void)hipEventDestroy(join[k]);
            st[k] = nullptr;
            join[k] = nullptr;
        }
        if (fork) (void)hipEventDestroy(fork);
        fork = nullptr;
    }
};

// ---- copies between device and caller memory ------------------------------
// Pinned staging shared by the read-outs and checkpoints of the process: a
// block as large as the small read-outs asked for, and a ring of slots that bulk
// copies go through while a few threads move finished slots to (from) the
// caller's pages, whose first touch is what a plain copy spends most of its
// time on.  Held while any simulation exists; a call that finds it in use by another
// thread copies without it.
constexpr size_t STAGE_SLOT = (size_t)4 << 20, STAGE_WORD = 256;
constexpr int STAGE_SLOTS = 8, STAGE_THREADS = 6;
// Parts up to this size are written to the block by a kernel: rho of 256^2 x 3
// (1.6 MB) takes 106 us so and 115 us through the ring, of 200^2 x 10 (3.2 MB)
// the ring.
constexpr size_t STAGE_SMALL_PART = STAGE_SLOT / 2;
// Bytes of bulk read-outs from which the ring is made.  Making it and giving it
// back costs 45 us and more (0.9 MB of populations read once 61 us plain, 103
// us with the ring; 2.6 MB 168 / 194; 4.9 MB 314 / 317; 14 MB 854 / 624), a
// plain copy 27 us a MB more than one through a ring that is there.
constexpr size_t STAGE_RING_FROM = STAGE_SLOT;
// Copies to the device go through it from this size: populations of 8.6 MB take
// 322 us to write so and 280 plain, 35 MB 1084 and 1113, 49 MB 1431 and 1706, 189
// MB 4554 and 6444.
constexpr size_t STAGE_WRITE_FROM = 9 * STAGE_SLOT;

struct Stage {
    std::mutex use;             // held by the call that copies through it
    char *block = nullptr;      // STAGE_WORD bytes for a status word, then data; pinned
    size_t block_bytes = 0;
    bool asked = false;         // a small read-out has done without the block
    size_t plain = 0;           // bytes of bulk read-outs that did without the ring
    char *ring = nullptr;       // STAGE_SLOTS * STAGE_SLOT, pinned
    hipEvent_t ev[STAGE_SLOTS] = {};
    std::mutex life;
    int sims = 0;               // live simulations
    Lanes lanes;

    char *slot(int64_t k) const { return ring + (k % STAGE_SLOTS) * STAGE_SLOT; }
    uint32_t *word() const { return (uint32_t *)block; }
    char *data() const { return block + STAGE_WORD; }
    static char *pinned(size_t bytes) {
        void *p = nullptr;
        if (hipHostMalloc(&p, bytes, 0) == hipSuccess) return (char *)p;
        (void)hipGetLastError();
        return nullptr;
    }
    // with `use` held: room for `bytes` of data in the block
    bool block_for(size_t bytes) {
        size_t want = (size_t)64 << 10;
        while (want < STAGE_WORD + bytes) want *= 2;
        if (want <= block_bytes) return true;
        if (block) (void)hipHostFree(block);
        block = pinned(want);
        block_bytes = block ? want : 0;
        return block != nullptr;
    }
    // with `use` held: the ring, where a read-out of `bytes` shall go through it
    bool ring_for(size_t bytes) {
        if (ring) return true;
        plain += bytes;
        if (plain < STAGE_RING_FROM) return false;
        for (hipEvent_t &e : ev)
            if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                e = nullptr;
                (void)hipGetLastError();
                return false;
            }
        ring = pinned(STAGE_SLOTS * STAGE_SLOT);
        return ring != nullptr;
    }
    void add_sim() {
        std::lock_guard<std::mutex> g(life);
        ++sims;
    }
    void drop_sim() {
        std::lock_guard<std::mutex> g(life);
        if (--sims > 0) return;
        lanes.release();
        std::lock_guard<std::mutex> u(use);
        if (block) (void)hipHostFree(block);
        if (ring) (void)hipHostFree(ring);
        block = ring = nullptr;
        block_bytes = plain = 0;
        asked = false;
        for (hipEvent_t &e : ev) {
            if (e) (void)hipEventDestroy(e);
            e = nullptr;
        }
    }
};

// That of the current device (one never destroyed, as simulations may outlive
// static objects).
Stage &device_stage() {
    static Stage *all = new Stage[64];
    int dev = 0;
    (void)hipGetDevice(&dev);
    return all[dev & 63];
}

// Copies `bytes` between the device (dev) and the caller (host) through the ring,
// on st, to the caller if `out`; done when it returns.  Slots are handed to the
// threads in order; none waits for anything but its own slot's turn, and all
// leave when the last slot is taken or a copy fails.
hipError_t staged_copy(Stage &g, char *host, char *dev, size_t bytes, bool out, hipStream_t st) {
    const int64_t n = (int64_t)((bytes + STAGE_SLOT - 1) / STAGE_SLOT);
    auto size = [&](int64_t k) { return std::min(STAGE_SLOT, bytes - (size_t)k * STAGE_SLOT); };
    auto host_at = [&](int64_t k) { return host + (size_t)k * STAGE_SLOT; };
    auto dev_at = [&](int64_t k) { return dev + (size_t)k * STAGE_SLOT; };
    auto dma = [&](int64_t k) {
        return out ? hipMemcpyAsync(g.slot(k), dev_at(k), size(k), hipMemcpyDeviceToHost, st)
                   : hipMemcpyAsync(dev_at(k), g.slot(k), size(k), hipMemcpyHostToDevice, st);
    };
    auto move = [&](int64_t k) {
        if (out)
            std::memcpy(host_at(k), g.slot(k), size(k));
        else
            std::memcpy(g.slot(k), host_at(k), size(k));
    };
    hipError_t err = hipSuccess;
    // a thread may take slot k once `open` > k; `moved` of the ring position
    // counts the slots that it has finished there
    std::atomic<int64_t> open{0}, next{0};
    std::atomic<int64_t> moved[STAGE_SLOTS];
    for (auto &m : moved) m.store(0);
    std::atomic<bool> stop{false};
    auto work = [&] {
        for (;;) {
            const int64_t k = next.fetch_add(1);
            if (k >= n) return;
            while (open.load(std::memory_order_acquire) <= k) {
                if (stop.load()) return;
                std::this_thread::yield();
            }
            move(k);
            moved[k % STAGE_SLOTS].fetch_add(1, std::memory_order_release);
        }
    };
    std::thread th[STAGE_THREADS];
    int nth = 0;
    if (n > 1) {
        try {
            for (; nth < STAGE_THREADS && nth < n; ++nth) th[nth] = std::thread(work);
        } catch (...) {
        }
    }
    if (nth == 0) {                        // one slot, or no thread to be had
        for (int64_t k = 0; k < n && err == hipSuccess; ++k) {
            if (!out) move(k);
            err = dma(k);
            if (err == hipSuccess) err = hipStreamSynchronize(st);
            if (out && err == hipSuccess) move(k);
        }
        return err;
    }
    auto finished = [&](int64_t k) {       // slot k's move is done
        return moved[k % STAGE_SLOTS].load(std::memory_order_acquire) > k / STAGE_SLOTS;
    };
    if (out) {
        int64_t issued = 0, landed = 0;
        while (landed < n && err == hipSuccess) {
            while (issued < n && issued < landed + STAGE_SLOTS && err == hipSuccess &&
                   (issued < STAGE_SLOTS || finished(issued - STAGE_SLOTS))) {
                err = dma(issued);
                if (err == hipSuccess) err = hipEventRecord(g.ev[issued % STAGE_SLOTS], st);
                ++issued;
            }
            if (err == hipSuccess && landed < issued) {
                err = hipEventSynchronize(g.ev[landed % STAGE_SLOTS]);
                ++landed;
                if (err == hipSuccess) open.store(landed, std::memory_order_release);
            } else {
                std::this_thread::yield();
            }
        }
    } else {
        open.store(std::min<int64_t>(n, STAGE_SLOTS));
        for (int64_t k = 0; k < n && err == hipSuccess; ++k) {
            while (!finished(k)) std::this_thread::yield();
            err = dma(k);
            if (err == hipSuccess) err = hipEventRecord(g.ev[k % STAGE_SLOTS], st);
            // the slot of the copy issued half a ring ago may be filled again
            const int64_t old = k - STAGE_SLOTS / 2;
            if (old >= 0 && err == hipSuccess) {
                err = hipEventSynchronize(g.ev[old % STAGE_SLOTS]);
                open.store(std::min<int64_t>(n, old + 1 + STAGE_SLOTS), std::memory_order_release);
            }
        }
        if (err == hipSuccess) err = hipStreamSynchronize(st);
    }
    if (err != hipSuccess) stop.store(true);
    for (int k = 0; k < nth; ++k) th[k].join();
    if (err != hipSuccess) (void)hipStreamSynchronize(st);
    return err;
}

// One part of a read-out: device to caller.
struct Part {
    void *host;
    const void *dev;
    size_t bytes;
};

// Copies the parts and the status word to the caller after the work queued
// on the simulation's stream; one wait in all where they are small.
fuglbm_status read_parts(fuglbm_sim *s, std::initializer_list<Part> parts) {
    hipStream_t st = s->last_stream;
    Stage &g = *s->stage;
    std::unique_lock<std::mutex> lk(g.use, std::try_to_lock);
    uint32_t word = 0;
    // (callers pass at most two parts)
    Part few[2] = {}, large[2] = {};
    int n = 0, nl = 0;
    for (const Part &p : parts)
        if (p.host) (p.bytes <= STAGE_SMALL_PART ? few[n++] : large[nl++]) = p;
    // making the block and giving it back costs as much (40 to 60 us) as it
    // spares the only small read-out of a simulation on its own: plain copies
    // first
    bool plain = !lk.owns_lock();
    if (!plain && !g.block && nl == 0 && !g.asked) plain = g.asked = true;
    if (plain || !g.block_for(few[0].bytes + few[1].bytes) ||
        (nl > 0 && !g.ring_for(large[0].bytes + large[1].bytes))) {
        HIP_TRY(hipStreamSynchronize(st));
        for (const Part &p : parts)
            if (p.host) HIP_TRY(hipMemcpy(p.host, p.dev, p.bytes, hipMemcpyDeviceToHost));
        HIP_TRY(hipMemcpy(&word, s->status, sizeof(word), hipMemcpyDeviceToHost));
        s->sticky |= word;
        return FUGLBM_OK;
    }
    // the large parts through the ring, the small ones and the status word by
    // one kernel and one wait
    if (n == 0 && nl > 0)
        HIP_TRY(hipMemcpyAsync(g.word(), s->status, sizeof(word), hipMemcpyDeviceToHost, st));
    for (int k = 0; k < nl; ++k)
        HIP_TRY(staged_copy(g, (char *)large[k].host, (char *)large[k].dev, large[k].bytes, true,
                            st));
    if (n > 0 || nl == 0)
        HIP_TRY(launch_to_host((const double *)few[0].dev, (int64_t)(few[0].bytes / 8),
                               (const double *)few[1].dev, (int64_t)(few[1].bytes / 8), s->status,
                               (double *)g.data(), g.word(), st));
    HIP_TRY(hipStreamSynchronize(st));
    for (int k = 0; k < n; ++k)
        std::memcpy(few[k].host, g.data() + (k ? few[0].bytes : 0), few[k].bytes);
    word = *g.word();
    s->sticky |= word;
    return FUGLBM_OK;
}

}  // namespace

extern "C" {

const char *fuglbm_last_error(void) { return g_err.c_str(); }

fuglbm_status fuglbm_init_mixture(const fuglbm_mixture_desc *d, fuglbm_mixture **out) {
    if (!d || !out) return fail(FUGLBM_EINVAL, "null argument");
    *out = nullptr;
    const int N = d->ncomp;
    if (N < 1 || N > FUGLBM_MAX_COMP) return fail(FUGLBM_EINVAL, "ncomp out of range");
    if (!d->Tc_K || !d->pc_bar || !d->omega || !d->M_gmol)
        return fail(FUGLBM_EINVAL, "null component array");
    if (d->ref_comp < 0 || d->ref_comp >= N) return fail(FUGLBM_EINVAL, "ref_comp out of range");
    if (d->eos < FUGLBM_EOS_PR || d->eos > FUGLBM_EOS_VDW) return fail(FUGLBM_EINVAL, "unknown eos");
    if (!(d->T_K > 0) || !std::isfinite(d->T_K)) return fail(FUGLBM_EINVAL, "T_K must be > 0");
    if (!(d->tau > 0.5) || !std::isfinite(d->tau)) return fail(FUGLBM_EINVAL, "tau must be > 1/2");
    if (!(d->kappa_ref_lu >= 0) || !std::isfinite(d->kappa_ref_lu))
        return fail(FUGLBM_EINVAL, "kappa_ref_lu must be >= 0");
    for (int i = 0; i < N; ++i) {
        if (!(d->Tc_K[i] > 0) || !(d->pc_bar[i] > 0) || !(d->M_gmol[i] > 0) ||
            !std::isfinite(d->omega[i]) || !std::isfinite(d->Tc_K[i]) ||
            !std::isfinite(d->pc_bar[i]) || !std::isfinite(d->M_gmol[i]))
            return fail(FUGLBM_EINVAL, "component constants must be positive and finite");
    }
    if (d->kij) {
        for (int i = 0; i < N; ++i) {
            if (d->kij[i * N + i] != 0.0) return fail(FUGLBM_EINVAL, "kij diagonal must be 0");
            for (int j = 0; j < N; ++j) {
                if (!std::isfinite(d->kij[i * N + j]) || d->kij[i * N + j] != d->kij[j * N + i])
                    return fail(FUGLBM_EINVAL, "kij must be finite and symmetric");
                if (!(d->kij[i * N + j] < 1.0)) return fail(FUGLBM_EINVAL, "kij must be < 1");
            }
        }
    }
    auto *m = new (std::nothrow) fuglbm_mixture();
    if (!m) return fail(FUGLBM_ENOMEM, "host allocation");
    const double a_ref = d->a_ref_lu > 0 ? d->a_ref_lu : 2.0 / 49.0;
    const double b_ref = d->b_ref_lu > 0 ? d->b_ref_lu : 2.0 / 21.0;
    const double R = d->R_lu > 0 ? d->R_lu : 1.0;
    const int c = d->ref_comp;
    const CubicEos E = cubic_eos(d->eos);
    // reference component's critical point in lattice units from a and b
    const double Tc_ref = (a_ref / b_ref) * (E.omega_b / E.omega_a) / R;
    const double pc_ref = E.omega_b * R * Tc_ref / b_ref;
    const double Tsc = Tc_ref / d->Tc_K[c];     // lattice units per K
    const double psc = pc_ref / d->pc_bar[c];   // lattice units per bar
    m->N = N;
    m->eos = d->eos;
    m->tau = d->tau;
    m->RT = R * d->T_K * Tsc;
    double a_lu[FUG_MAXC];
    for (int i = 0; i < N; ++i) {
        const double Tc = d->Tc_K[i] * Tsc, pc = d->pc_bar[i] * psc;
        a_lu[i] = E.omega_a * R * R * Tc * Tc / pc;
        m->b[i] = E.omega_b * R * Tc / pc;
        m->aa[i] = a_lu[i] * cubic_alpha(d->eos, d->omega[i], d->T_K / d->Tc_K[i]);
        m->M[i] = d->M_gmol[i] / d->M_gmol[c];
    }
    for (int i = 0; i < N; ++i) {
        m->sqk[i] = std::sqrt(d->kappa_ref_lu * a_lu[i] / a_lu[c]);
        for (int j = 0; j < N; ++j) {
            const double k = d->kij ? d->kij[i * N + j] : 0.0;
            m->aij[i * FUG_MAXC + j] = std::sqrt(m->aa[i] * m->aa[j]) * (1.0 - k);
        }
    }
    *out = m;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_lattice_constants(const fuglbm_mixture *m, double *out, size_t n) {
    if (!m || !out) return fail(FUGLBM_EINVAL, "null argument");
    const int N = m->N;
    if (n < (size_t)(1 + 4 * N + N * N)) return fail(FUGLBM_EINVAL, "output too small");
    size_t k = 0;
    out[k++] = m->RT;
    for (int i = 0; i < N; ++i) {
        out[k++] = m->b[i];
        out[k++] = m->aa[i];
        out[k++] = m->sqk[i];
        out[k++] = m->M[i];
    }
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) out[k++] = m->aij[i * FUG_MAXC + j];
    return FUGLBM_OK;
}

void fuglbm_destroy_mixture(fuglbm_mixture *m) { delete m; }

size_t fuglbm_fields_bytes(int32_t ncomp, fuglbm_lattice lattice, fuglbm_precision prec,
                           int32_t nx, int32_t ny, int32_t nz) {
    if (ncomp < 1 || ncomp > FUGLBM_MAX_COMP || nx < 1 || ny < 1 || nz < 1) return 0;
    if (lattice != FUGLBM_D2Q9 && lattice != FUGLBM_D3Q19) return 0;
    return carve(ncomp, lattice, prec == FUGLBM_FP32_STORAGE, nx, ny, nz).total;
}

fuglbm_status fuglbm_init_fields(const fuglbm_mixture *mix, fuglbm_lattice lattice,
                                 fuglbm_precision prec, int32_t nx, int32_t ny, int32_t nz,
                                 const double *rho, void *dev_buf, void *hip_stream,
                                 fuglbm_sim **out) {
    const TraceRange trace_range("fuglbm_init_fields");
    if (!mix || !rho || !out) return fail(FUGLBM_EINVAL, "null argument");
    *out = nullptr;
    if (lattice != FUGLBM_D2Q9 && lattice != FUGLBM_D3Q19) return fail(FUGLBM_EINVAL, "lattice");
    if (prec != FUGLBM_FP64 && prec != FUGLBM_FP32_STORAGE) return fail(FUGLBM_EINVAL, "precision");
    if (nx < 1 || ny < 1 || nz < 1) return fail(FUGLBM_EINVAL, "grid sizes must be >= 1");
    if (lattice == FUGLBM_D2Q9 && nz != 1) return fail(FUGLBM_EINVAL, "D2Q9 needs nz == 1");
    const int64_t ns = (int64_t)nx * ny * nz;
    if (ns > (int64_t)1 << 31) return fail(FUGLBM_EINVAL, "grid too large");
    const int N = mix->N;
    // physical admissibility of the initial field (rho_i > 0, finite, b_m rt < 1)
    for (int64_t s = 0; s < ns; ++s) {
        double eta = 0.0;
        for (int i = 0; i < N; ++i) {
            const double r = rho[(int64_t)i * ns + s];
            if (!std::isfinite(r) || !(r > 0.0))
                return fail(FUGLBM_EUNPHYSICAL, "rho_i must be finite and > 0");
            eta += mix->b[i] * r / mix->M[i];
        }
        if (!(eta < 1.0)) return fail(FUGLBM_EUNPHYSICAL, "b_m * rt >= 1 (outside the EOS domain)");
    }
    auto *s = new (std::nothrow) fuglbm_sim();
    if (!s) return fail(FUGLBM_ENOMEM, "host allocation");
    s->mix = mix;
    s->lattice = lattice;
    s->fp32 = prec == FUGLBM_FP32_STORAGE;
    s->nx = nx; s->ny = ny; s->nz = nz;
    s->N = N;
    s->Q = lattice_Q(lattice);
    s->D = lattice_D(lattice);
    s->ns = ns;
    s->cv = carve(N, lattice, s->fp32, nx, ny, nz);
    hipStream_t st = (hipStream_t)hip_stream;
    s->last_stream = st;
    if (dev_buf) {
        if (((uintptr_t)dev_buf & 255) != 0) {
            delete s;
            return fail(FUGLBM_EINVAL, "dev_buf must be 256-byte aligned");
        }
        s->base = (char *)dev_buf;
        s->owned = false;
    } else {
        void *p = nullptr;
        hipError_t e = hipMalloc(&p, s->cv.total);
        if (e != hipSuccess) {
            delete s;
            return fail(FUGLBM_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
        }
        s->base = (char *)p;
        s->owned = true;
    }
    s->buf[0] = s->base + s->cv.buf0;
    s->buf[1] = s->base + s->cv.buf1;
    s->dc = (SimConst *)(s->base + s->cv.cst);
    s->status = (uint32_t *)(s->base + s->cv.status);
    s->rho_f = (double *)(s->base + s->cv.rho);
    s->psi_f = (double *)(s->base + s->cv.psi);
    s->s_f = (double *)(s->base + s->cv.s);
    s->j_f = (double *)(s->base + s->cv.j);
    s->u_f = (double *)(s->base + s->cv.u);
    s->snap = (double *)(s->base + s->cv.snap);
    s->part = (double *)(s->base + s->cv.part);
    s->fsim = (FusedSim *)(s->base + s->cv.fsim);
    s->items = (FusedItem *)(s->base + s->cv.items);
    s->parity = 0;
    if (hipEventCreateWithFlags(&s->done, hipEventDisableTiming) != hipSuccess) {
        if (s->owned) (void)hipFree(s->base);
        delete s;
        return fail(FUGLBM_EDEVICE, "hipEventCreate");
    }
    s->done_valid = false;
    // constant block
    SimConst &c = s->hc;
    std::memset(&c, 0, sizeof(c));
    c.N = N;
    c.lattice = lattice;
    c.nx = nx; c.ny = ny; c.nz = nz;
    c.nsites = ns;
    c.omega = 1.0 / mix->tau;
    c.fcoef = 1.0 - 1.0 / (2.0 * mix->tau);
    c.RT = mix->RT;
    c.invRT = 1.0 / mix->RT;
    {
        const CubicEos E = cubic_eos(mix->eos);
        c.eos = mix->eos;
        c.d1 = E.d1;
        c.d2 = E.d2;
        c.eu = E.u;
        c.ew = E.w;
        c.dk = mix->eos == FUGLBM_EOS_VDW ? 0.0 : 1.0 / (E.d1 - E.d2);
    }
    for (int i = 0; i < N; ++i) {
        c.b[i] = mix->b[i];
        c.M[i] = mix->M[i];
        c.invM[i] = 1.0 / mix->M[i];
        c.sqk[i] = mix->sqk[i];
        for (int j = 0; j < N; ++j) c.aij[i * FUG_MAXC + j] = mix->aij[i * FUG_MAXC + j];
    }
    fuglbm_status rc = FUGLBM_OK;
    auto bail = [&](fuglbm_status r) {
        (void)hipEventDestroy(s->done);
        if (s->owned) (void)hipFree(s->base);
        delete s;
        return r;
    };
    hipError_t e = hipMemcpy(s->dc, &c, sizeof(SimConst), hipMemcpyHostToDevice);
    if (e != hipSuccess) return bail(hip_fail(e, "upload constants"));
    // stage rho in the second population buffer, then g = geq(rho, u = 0)
    e = hipMemcpy(s->buf[1], rho, (size_t)N * ns * sizeof(double), hipMemcpyHostToDevice);
    if (e != hipSuccess) return bail(hip_fail(e, "upload rho"));
    e = hipMemset(s->status, 0, 256);
    if (e != hipSuccess) return bail(hip_fail(e, "clear status"));
    e = launch_init(lattice, s->fp32, s->dc, ns, (const double *)s->buf[1], s->buf[0], st);
    if (e != hipSuccess) return bail(hip_fail(e, "init kernel"));
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return bail(hip_fail(e, "init sync"));
    // fused-kernel tables (D2Q9)
    const FusedSim fs = fused_sim(s);
    e = hipMemcpy(s->fsim, &fs, sizeof(FusedSim), hipMemcpyHostToDevice);
    if (e != hipSuccess) return bail(hip_fail(e, "upload fused sim"));
    const bool fused = fused_fits(s);
    s->kernel = default_kernel(s);
    s->rows = fused ? auto_rows(nx, ny, N, s->fp32, s->kernel) : 0;
    s->auto_kernel = fused;
    if (fused) {
        rc = build_items(s);
        if (rc != FUGLBM_OK) return bail(rc);
    }
    s->step = 0;
    s->snap_step = 0;
    s->have_snap = false;
    s->sticky = 0;
    s->autotune = fused;
    s->tuned = false;
    s->form = s->taken = FUGLBM_FORM_AUTO;
    s->form_rows = 0;
    s->fgraph[0] = s->fgraph[1] = nullptr;
    s->uid = next_sim_uid();
    s->stage = &device_stage();
    s->stage->add_sim();
    *out = s;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_get_tuning(const fuglbm_sim *s, int32_t *kernel, int32_t *rows) {
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    if (kernel) *kernel = s->kernel;
    if (rows) *rows = is_fused(s->kernel) ? s->rows : 0;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_set_tuning(fuglbm_sim *s, int32_t kernel, int32_t rows) {
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    if (kernel < 0 || kernel > 3) return fail(FUGLBM_EINVAL, "kernel must be 0, 1, 2 or 3");
    if (is_fused(kernel) && !fused_fits(s))
        return fail(FUGLBM_EINVAL, "the fused kernel is D2Q9 only, with < 2^32 elements per buffer");
    if (kernel == 3 && !ws_usable(s->N, s->fp32))
        return fail(FUGLBM_EINVAL, "the store-wave fused kernel is built for at most 10 components");
    if (rows < 0) return fail(FUGLBM_EINVAL, "rows must be >= 0");
    const int k = kernel == 0 ? default_kernel(s) : kernel;
    s->auto_kernel = kernel == 0 && is_fused(k);
    int r = s->rows;
    if (is_fused(k)) {
        r = rows == 0 ? auto_rows(s->nx, s->ny, s->N, s->fp32, k) : std::min<int>(rows, s->ny);
        s->autotune = rows == 0;
        s->tuned = false;
    }
    HIP_TRY(hipStreamSynchronize(s->last_stream));
    s->uid = next_sim_uid();   // batch tables hold what was chosen before
    s->kernel = k;
    s->form = kernel ? FUGLBM_FORM_POPULATIONS : FUGLBM_FORM_AUTO;
    if (r != s->rows) {
        s->rows = r;
        fuglbm_status rc = build_items(s);
        if (rc != FUGLBM_OK) return rc;
    }
    drop_graphs(s);
    return FUGLBM_OK;
}

fuglbm_status fuglbm_set_form(fuglbm_sim *s, int32_t form) {
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    const bool single = form == FUGLBM_FORM_FIELDS_SINGLE;
    if (form < FUGLBM_FORM_AUTO || form > FUGLBM_FORM_FIELDS_SINGLE)
        return fail(FUGLBM_EINVAL, "unknown form");
    if (form >= FUGLBM_FORM_FIELDS && !field_fits(s) &&
        (single || !field3_fits(s) || field3_shape(s).cost == Shape3::NONE))
        return fail(FUGLBM_EINVAL, "the simulation's steps have no such form");
    if (single && s->N > field_single_comp())
        return fail(FUGLBM_EINVAL, "steps by single wavefronts are built for at most 3 components");
    HIP_TRY(hipStreamSynchronize(s->last_stream));
    s->uid = next_sim_uid();
    drop_graphs(s);
    s->form = form;
    s->form_rows = form_fixed(s) && is_fused(s->kernel)
                       ? (s->autotune ? field_model_rows({s}, single) : s->rows)
                       : 0;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_get_form(const fuglbm_sim *s, int32_t *form) {
    if (!s || !form) return fail(FUGLBM_EINVAL, "null argument");
    *form = s->taken;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_sim_info(const fuglbm_sim *s, int32_t *Q, int32_t *D, int64_t *sites,
                              int64_t *alg_bytes, int32_t *kernel) {
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    if (Q) *Q = s->Q;
    if (D) *D = s->D;
    if (sites) *sites = s->ns;
    // algorithmic bytes: every population read and written once (no padding)
    if (alg_bytes) *alg_bytes = 2 * (int64_t)s->N * s->ns * (8 + (s->Q - 1) * (s->fp32 ? 4 : 8));
    if (kernel) *kernel = s->kernel;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_step_n(fuglbm_sim *s, int64_t nsteps, void *hip_stream) {
    const TraceRange trace_range("fuglbm_step_n");
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    if (nsteps < 0) return fail(FUGLBM_EINVAL, "nsteps must be >= 0");
    if (s->sticky) return fail(FUGLBM_ENONFINITE, "simulation has a sticky device error");
    hipStream_t st = (hipStream_t)hip_stream;
    {
        fuglbm_status rc = order_after(s, st);
        if (rc != FUGLBM_OK) return rc;
    }
    int64_t left = nsteps;
    if (left == 0) return mark_done(s, st);
    const bool fixed = form_fixed(s) && field_fits(s);
    if (is_fused(s->kernel) && s->autotune && !s->tuned && !fixed) {
        fuglbm_status rc = autotune_rows(s, st);
        if (rc != FUGLBM_OK) return rc;
    }
    // (a stream that the caller captures cannot be timed)
    if (left >= 2 && s->tuned && field_usable(s) && !s->tune.frows && !capturing(st)) {
        fuglbm_status rc = autotune_field(s, st);
        if (rc != FUGLBM_OK) return rc;
    }
    if (fixed || (s->tuned && field_usable(s) && field_pays(s->tune, left))) {
        const int rows = fixed ? s->form_rows : s->tune.frows;
        const bool single = fixed ? s->form == FUGLBM_FORM_FIELDS_SINGLE : s->tune.single;
        fuglbm_status rc = run_field(field_run(s, rows, single), s->N, s->fp32, left,
                                     s->fgraph[s->parity], st);
        if (rc != FUGLBM_OK) return rc;
        s->step += left;
        s->taken = single ? FUGLBM_FORM_FIELDS_SINGLE : FUGLBM_FORM_FIELDS;
        return mark_done(s, st);
    }
    if (field3_alone(s, left)) {
        fuglbm_status rc = run_field3(s, left, st);
        if (rc != FUGLBM_OK) return rc;
        return mark_done(s, st);
    }
    s->taken = FUGLBM_FORM_POPULATIONS;
    // odd parity first so that graph replays start from buffer 0
    if (left > 0 && s->parity == 1 && left >= 2 * GRAPH_STEPS) {
        hipError_t e = launch_one_step(s, s->parity, st);
        if (e != hipSuccess) return hip_fail(e, "step launch");
        s->parity ^= 1;
        --left;
        ++s->step;
    }
    if (left >= 2 * GRAPH_STEPS && s->parity == 0) {
        fuglbm_status rc = ensure_graph(s);
        if (rc != FUGLBM_OK) return rc;
        while (left >= GRAPH_STEPS) {
            HIP_TRY(hipGraphLaunch(s->graph.exec, st));
            left -= GRAPH_STEPS;
            s->step += GRAPH_STEPS;
        }
    }
    for (; left > 0; --left) {
        hipError_t e = launch_one_step(s, s->parity, st);
        if (e != hipSuccess) return hip_fail(e, "step launch");
        s->parity ^= 1;
        ++s->step;
    }
    return mark_done(s, st);
}

fuglbm_status fuglbm_read_moments(fuglbm_sim *s, double *rho_out, double *u_out,
                                  fuglbm_diag *diag) {
    const TraceRange trace_range("fuglbm_read_moments");
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    hipStream_t st = s->last_stream;
    HIP_TRY(launch_fields(s->lattice, s->fp32, s->dc, s->nx, s->ny, s->nz, s->buf[s->parity],
                          s->rho_f, s->psi_f, s->s_f, s->j_f, u_out ? s->u_f : nullptr, s->status,
                          st));
    fuglbm_status rc = read_parts(s, {{rho_out, s->rho_f, (size_t)s->N * s->ns * 8},
                                      {u_out, s->u_f, (size_t)s->D * s->ns * 8}});
    if (rc != FUGLBM_OK) return rc;
    if (diag) {
        rc = fuglbm_diagnostics(s, diag);
        if (rc != FUGLBM_OK && rc != FUGLBM_ENONFINITE) return rc;
    }
    if (s->sticky) return fail(FUGLBM_ENONFINITE, "device status bits set");
    return FUGLBM_OK;
}

// Diagnostics: the fields pass (rho_i, j, force-corrected u of the current
// state), then per-block partial sums and one fixed-order final sum per
// quantity on the device; the host reads the (N + 1) x DIAG_QUANT totals.
fuglbm_status fuglbm_diagnostics(fuglbm_sim *s, fuglbm_diag *diag) {
    const TraceRange trace_range("fuglbm_diagnostics");
    if (!s || !diag) return fail(FUGLBM_EINVAL, "null argument");
    hipStream_t st = s->last_stream;
    const int nblk = diag_blocks(s->ns);
    const int N = s->N;
    double *fin = s->part + (size_t)1024 * (N + 1) * DIAG_QUANT;
    HIP_TRY(launch_fields(s->lattice, s->fp32, s->dc, s->nx, s->ny, s->nz, s->buf[s->parity],
                          s->rho_f, s->psi_f, s->s_f, s->j_f, s->u_f, s->status, st));
    HIP_TRY(launch_diag(s->D, N, s->ns, s->rho_f, s->j_f, s->u_f, s->snap, s->part, nblk, fin,
                        s->have_snap ? 1 : 0, st));
    double tot[(FUGLBM_MAX_COMP + 1) * DIAG_QUANT];
    fuglbm_status rc = read_parts(s, {{tot, fin, sizeof(double) * (N + 1) * DIAG_QUANT}});
    if (rc != FUGLBM_OK) return rc;
    std::memset(diag, 0, sizeof(*diag));
    diag->step = s->step;
    for (int i = 0; i < N; ++i) diag->mass[i] = tot[i * DIAG_QUANT];
    for (int d = 0; d < s->D; ++d) {
        diag->momentum_pop[d] = tot[N * DIAG_QUANT + d];
        diag->momentum[d] = tot[N * DIAG_QUANT + 3 + d];
    }
    double res = 0.0;
    const int64_t K = s->step - s->snap_step;
    if (s->have_snap && K > 0)
        for (int i = 0; i < N; ++i)
            res = std::max(res, tot[i * DIAG_QUANT + 1] / ((double)K * tot[i * DIAG_QUANT]));
    diag->residual = res;
    s->have_snap = true;
    s->snap_step = s->step;
    diag->status = s->sticky;
    if (s->sticky) return fail(FUGLBM_ENONFINITE, "device status bits set");
    return FUGLBM_OK;
}

extern "C++" {
// Column of the stored moving population a of column x (pop_col).
static int host_pop_col(const fuglbm_sim *s, int a, int x) {
    return s->lattice == FUGLBM_D3Q19 ? pop_col<D3Q19>(a, x, s->nx) : pop_col<D2Q9>(a, x, s->nx);
}

}  // extern "C++"

// Checkpoint and restore: the device orders the populations as the host
// array has them (planes [N][Q][sites] FP64, as many at a time as fit the
// scratch buffer: all of them in FP64, at least five of FP32 storage), and
// whole planes are copied.
extern "C++" {
template <class Fn>
static fuglbm_status for_planes(const fuglbm_sim *s, Fn fn) {
    const int total = s->N * s->Q;
    const int most = (int)std::min<int64_t>(total, pop_bytes(s) / (s->ns * 8));
    for (int p = 0; p < total; p += most) {
        const fuglbm_status rc = fn(p, std::min(most, total - p));
        if (rc != FUGLBM_OK) return rc;
    }
    return FUGLBM_OK;
}

// Up to this many bytes of populations the host orders them: a launch and a
// wait take as long (0.22 MB 22 us to read and 21 to write, ordered by the
// device 31 and 31; 0.88 MB 66 and 57, 58 and 55).
constexpr int64_t HOST_ORDER = 512 << 10;
static bool host_orders(const fuglbm_sim *s) { return (int64_t)s->N * s->Q * s->ns * 8 <= HOST_ORDER; }

// Host copy `buf` of a population buffer -> g (OUT) or back.
template <typename ST, bool OUT, class G>
static void order_pops(const fuglbm_sim *s, char *buf, G *g) {
    const int64_t rows = (int64_t)s->ny * s->nz;
    const PopLayout<ST> P(s->N, s->Q, s->nx, rows);
    for (int i = 0; i < s->N; ++i)
        for (int a = 0; a < s->Q; ++a)
            for (int64_t r = 0; r < rows; ++r) {
                G *o = g + ((size_t)i * s->Q + a) * s->ns + (size_t)r * s->nx;
                double *rest = (double *)(buf + P.rest(r, i, 0));
                ST *move = a ? (ST *)(buf + P.move(r, i, a, 0)) : nullptr;
                for (int x = 0; x < s->nx; ++x) {
                    if constexpr (OUT)
                        o[x] = a ? (double)move[host_pop_col(s, a, x)] : rest[x];
                    else if (a)
                        move[host_pop_col(s, a, x)] = (ST)o[x];
                    else
                        rest[x] = o[x];
                }
            }
}
}  // extern "C++"

fuglbm_status fuglbm_read_populations(fuglbm_sim *s, double *g_out) {
    if (!s || !g_out) return fail(FUGLBM_EINVAL, "null argument");
    hipStream_t st = s->last_stream;
    if (host_orders(s)) {
        std::unique_ptr<char[]> tmp(new (std::nothrow) char[(size_t)pop_bytes(s)]);
        if (!tmp) return fail(FUGLBM_ENOMEM, "host allocation");
        HIP_TRY(hipStreamSynchronize(st));
        HIP_TRY(hipMemcpy(tmp.get(), s->buf[s->parity], (size_t)pop_bytes(s),
                          hipMemcpyDeviceToHost));
        s->fp32 ? order_pops<float, true>(s, tmp.get(), g_out)
                : order_pops<double, true>(s, tmp.get(), g_out);
        return FUGLBM_OK;
    }
    // the spare buffer is what the next step overwrites
    char *scratch = (char *)s->buf[s->parity ^ 1];
    Stage &g = *s->stage;
    std::unique_lock<std::mutex> lk(g.use, std::try_to_lock);
    const bool staged = lk.owns_lock() && g.ring_for((size_t)s->N * s->Q * s->ns * 8);
    return for_planes(s, [&](int p, int n) -> fuglbm_status {
        char *host = (char *)(g_out + (size_t)p * s->ns);
        const size_t bytes = (size_t)n * s->ns * 8;
        HIP_TRY(launch_planes(s->lattice, s->fp32, true, s->N, s->nx, s->ny, s->nz, p, n,
                              s->buf[s->parity], scratch, st));
        if (staged) {
            HIP_TRY(staged_copy(g, host, scratch, bytes, true, st));
        } else {
            HIP_TRY(hipStreamSynchronize(st));
            HIP_TRY(hipMemcpy(host, scratch, bytes, hipMemcpyDeviceToHost));
        }
        return FUGLBM_OK;
    });
}

fuglbm_status fuglbm_write_populations(fuglbm_sim *s, const double *g_in, int64_t step) {
    if (!s || !g_in) return fail(FUGLBM_EINVAL, "null argument");
    if (step < 0) return fail(FUGLBM_EINVAL, "step must be >= 0");
    hipStream_t st = s->last_stream;
    HIP_TRY(hipStreamSynchronize(st));
    if (host_orders(s)) {
        // (zeros in what the layout pads)
        std::unique_ptr<char[]> tmp(new (std::nothrow) char[(size_t)pop_bytes(s)]());
        if (!tmp) return fail(FUGLBM_ENOMEM, "host allocation");
        s->fp32 ? order_pops<float, false>(s, tmp.get(), g_in)
                : order_pops<double, false>(s, tmp.get(), g_in);
        HIP_TRY(hipMemcpy(s->buf[0], tmp.get(), (size_t)pop_bytes(s), hipMemcpyHostToDevice));
    } else {
        char *scratch = (char *)s->buf[1];
        Stage &g = *s->stage;
        const size_t all = (size_t)s->N * s->Q * s->ns * 8;
        std::unique_lock<std::mutex> lk(g.use, std::defer_lock);
        const bool staged = all >= STAGE_WRITE_FROM && lk.try_lock() && g.ring_for(all);
        fuglbm_status rc = for_planes(s, [&](int p, int n) -> fuglbm_status {
            char *host = (char *)(g_in + (size_t)p * s->ns);
            const size_t bytes = (size_t)n * s->ns * 8;
            if (staged)
                HIP_TRY(staged_copy(g, host, scratch, bytes, false, st));
            else
                HIP_TRY(hipMemcpy(scratch, host, bytes, hipMemcpyHostToDevice));
            HIP_TRY(launch_planes(s->lattice, s->fp32, false, s->N, s->nx, s->ny, s->nz, p, n,
                                  s->buf[0], scratch, st));
            HIP_TRY(hipStreamSynchronize(st));
            return FUGLBM_OK;
        });
        if (rc != FUGLBM_OK) return rc;
    }
    s->parity = 0;
    s->step = step;
    s->have_snap = false;
    return FUGLBM_OK;
}

fuglbm_status fuglbm_poke_population(fuglbm_sim *s, int32_t comp, int32_t a, int64_t site,
                                     double value) {
    if (!s) return fail(FUGLBM_EINVAL, "null sim");
    if (comp < 0 || comp >= s->N || a < 0 || a >= s->Q || site < 0 || site >= s->ns)
        return fail(FUGLBM_EINVAL, "index out of range");
    HIP_TRY(hipStreamSynchronize(s->last_stream));
    const int64_t row = site / s->nx;
    const int x = (int)(site - row * s->nx);
    char *b = (char *)s->buf[s->parity];
    if (a == 0) {
        const int64_t off = s->fp32 ? PopLayout<float>(s->N, s->Q, s->nx, (int64_t)s->ny * s->nz).rest(row, comp, x)
                                    : PopLayout<double>(s->N, s->Q, s->nx, (int64_t)s->ny * s->nz).rest(row, comp, x);
        HIP_TRY(hipMemcpy(b + off, &value, 8, hipMemcpyHostToDevice));
    } else if (s->fp32) {
        const float f = (float)value;
        const int64_t off = PopLayout<float>(s->N, s->Q, s->nx, (int64_t)s->ny * s->nz).move(row, comp, a, host_pop_col(s, a, x));
        HIP_TRY(hipMemcpy(b + off, &f, 4, hipMemcpyHostToDevice));
    } else {
        const int64_t off = PopLayout<double>(s->N, s->Q, s->nx, (int64_t)s->ny * s->nz).move(row, comp, a, host_pop_col(s, a, x));
        HIP_TRY(hipMemcpy(b + off, &value, 8, hipMemcpyHostToDevice));
    }
    return FUGLBM_OK;
}

extern "C++" {
static void forget_sim_in_batches(const fuglbm_sim *s);
}

void fuglbm_destroy_sim(fuglbm_sim *s) {
    if (!s) return;
    (void)hipStreamSynchronize(s->last_stream);
    forget_sim_in_batches(s);
    drop_graphs(s);
    if (s->done) (void)hipEventDestroy(s->done);
    if (s->owned) (void)hipFree(s->base);
    s->stage->drop_sim();
    delete s;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Batched stepping: D2Q9 simulations on the fused kernel that share the
// component count and precision run as ONE launch per step over a combined
// work-item table; the table is rebuilt only when the set of simulations
// (or their buffer parities, or the tuning that a caller set) changes.
// ---------------------------------------------------------------------------
namespace {

struct BatchTable {
    std::vector<fuglbm_sim *> sims;
    std::vector<uint64_t> uids;
    std::vector<int> parity0;
    FusedSim *dsims = nullptr;
    FusedItem *ditems = nullptr;
    size_t cap_sims = 0, cap_items = 0;
    int nitems = 0;
    int kernel = 2;                   // fused variant of the launches
    int rows = 0;                     // most rows of an item
    hipGraphExec_t graph = nullptr;   // GRAPH_STEPS launches starting at flip 0
    // field form: its member and item tables, what the tuner measured, and a
    // graph per flip
    FieldSim *dfield = nullptr;
    FusedItem *dfitems = nullptr;
    size_t cap_fsims = 0, cap_fitems = 0;
    FieldRun frun{};
    Tuned tune;
    hipGraphExec_t fgraph[2] = {nullptr, nullptr};
    hipStream_t last_stream = nullptr;
    bool used = false;                // last_stream is meaningful

    FusedTable table() const { return {ditems, nitems, dsims, (int)sims.size(), rows}; }
};

fuglbm_status batch_graph(BatchTable &bt, int ncomp, bool fp32) {
    if (bt.graph) return FUGLBM_OK;
    return capture_steps(
        [&](int k, hipStream_t cs) {
            return launch_fused(bt.kernel, ncomp, fp32, bt.table(), k & 1, cs);
        },
        bt.graph, "batch graph");
}

void drop_batch_graphs(BatchTable &bt) {
    for (hipGraphExec_t *g : {&bt.graph, &bt.fgraph[0], &bt.fgraph[1]}) {
        if (*g) (void)hipGraphExecDestroy(*g);
        *g = nullptr;
    }
}

// By component count, precision, the form that the members' callers fixed
// (AUTO where none did), and 1 or 2 for the halves of a group that is split.
using BatchKey = std::tuple<int, int, int, int>;
std::map<BatchKey, BatchTable> &batch_tables() {
    static std::map<BatchKey, BatchTable> t;
    return t;
}

// Items in logical order -> launch order: workgroups are handed to the 8
// XCDs round-robin, XCD k gets the k-th contiguous slice.
std::vector<FusedItem> deal_items(const std::vector<FusedItem> &logical) {
    const int n = (int)logical.size();
    const int per = (n + 7) / 8;
    std::vector<FusedItem> items((size_t)per * 8, FusedItem{-1, 0, 0, 0});
    for (int b = 0; b < per * 8; ++b) {
        const int li = (b % 8) * per + b / 8;
        if (li < n) items[b] = logical[li];
    }
    return items;
}

// Device array of at least n elements; a growing one doubles.
template <class T>
fuglbm_status grow(T *&p, size_t &cap, size_t n) {
    if (n <= cap) return FUGLBM_OK;
    if (p) (void)hipFree(p);
    p = nullptr;
    cap = 0;
    HIP_TRY(hipMalloc(&p, 2 * n * sizeof(T)));
    cap = 2 * n;
    return FUGLBM_OK;
}

// The field form's tables for a group at `rows` rows per item -> bt.frun.
fuglbm_status build_field_batch(BatchTable &bt, const std::vector<fuglbm_sim *> &group, int rows,
                                hipStream_t st) {
    HIP_TRY(hipStreamSynchronize(st));  // the old tables may still be read
    std::vector<FieldSim> fs;
    std::vector<FusedItem> logical;
    int64_t blocks = 0;
    for (size_t k = 0; k < group.size(); ++k) {
        const fuglbm_sim *s = group[k];
        fs.push_back(field_sim(s));
        fs.back().end = blocks += (s->ns + 255) / 256;
        const int strips = (s->nx + FUSED_OUT - 1) / FUSED_OUT, rw = std::min(rows, s->ny);
        for (int y = 0; y < s->ny; y += rw)
            for (int x = 0; x < strips; ++x)
                logical.push_back({(int32_t)k, x * FUSED_OUT, y, std::min(rw, s->ny - y)});
    }
    if (blocks > INT32_MAX) return fail(FUGLBM_EINVAL, "batch too large for one launch");
    const std::vector<FusedItem> items = deal_items(logical);
    fuglbm_status rc = grow(bt.dfield, bt.cap_fsims, fs.size());
    if (rc == FUGLBM_OK) rc = grow(bt.dfitems, bt.cap_fitems, items.size());
    if (rc != FUGLBM_OK) return rc;
    HIP_TRY(hipMemcpy(bt.dfield, fs.data(), fs.size() * sizeof(FieldSim), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(bt.dfitems, items.data(), items.size() * sizeof(FusedItem),
                      hipMemcpyHostToDevice));
    bt.frun = FieldRun{};
    bt.frun.tab = bt.dfield;
    bt.frun.nm = (int)fs.size();
    bt.frun.items = bt.dfitems;
    bt.frun.nitems = (int)items.size();
    bt.frun.blocks = blocks;
    return FUGLBM_OK;
}

// rows > 0: every member uses min(rows, ny) rows per item; 0: its own.
// kernel: the fused variant (0: that of the first member).
fuglbm_status build_batch(BatchTable &bt, const std::vector<fuglbm_sim *> &group, hipStream_t st,
                          int rows = 0, int kernel = 0) {
    HIP_TRY(hipStreamSynchronize(st));  // the old table may still be read by queued launches
    drop_batch_graphs(bt);
    bt.kernel = kernel ? kernel : group[0]->kernel;
    bt.rows = 0;
    std::vector<FusedSim> hs;
    std::vector<FusedItem> logical;
    for (size_t k = 0; k < group.size(); ++k) {
        fuglbm_sim *s = group[k];
        hs.push_back(fused_sim(s));
        const int strips = (s->nx + FUSED_OUT - 1) / FUSED_OUT;
        const int rw = rows > 0 ? std::min(rows, s->ny) : s->rows;
        bt.rows = std::max(bt.rows, rw);
        const int chunks = (s->ny + rw - 1) / rw;
        for (int c = 0; c < chunks; ++c)
            for (int t = 0; t < strips; ++t)
                logical.push_back({(int32_t)k, t * FUSED_OUT, c * rw, std::min(rw, s->ny - c * rw)});
    }
    const std::vector<FusedItem> items = deal_items(logical);
    if (hs.size() > bt.cap_sims) {
        if (bt.dsims) (void)hipFree(bt.dsims);
        bt.cap_sims = hs.size() * 2;
        HIP_TRY(hipMalloc(&bt.dsims, bt.cap_sims * sizeof(FusedSim)));
    }
    if (items.size() > bt.cap_items) {
        if (bt.ditems) (void)hipFree(bt.ditems);
        bt.cap_items = items.size() * 2;
        HIP_TRY(hipMalloc(&bt.ditems, bt.cap_items * sizeof(FusedItem)));
    }
    HIP_TRY(hipMemcpy(bt.dsims, hs.data(), hs.size() * sizeof(FusedSim), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(bt.ditems, items.data(), items.size() * sizeof(FusedItem),
                      hipMemcpyHostToDevice));
    bt.nitems = (int)items.size();
    bt.sims = group;
    bt.uids.clear();
    for (auto *sp : group) bt.uids.push_back(sp->uid);
    bt.parity0.clear();
    for (auto *s : group) bt.parity0.push_back(s->parity);
    return FUGLBM_OK;
}

// Batched launches: the rows-per-item autotuner over one uniform rows value
// for all members, cached per batch class: component count, precision, and
// the power-of-two classes of the total strip-rows (strips x ny summed over
// members, which sets the item count against the resident slots) and of the
// tallest member.  Batches of a serving loop change members often; a class
// key lets them reuse one tuning.  Leaves bt built with the chosen rows.
static int log2_class(int64_t v) {
    int k = 0;
    while (v > 1) {
        v >>= 1;
        ++k;
    }
    return k;
}

using BatchClass = std::tuple<int, int, int, int>;
std::map<BatchClass, Tuned> &batch_tune_cache() {
    static std::map<BatchClass, Tuned> m;
    return m;
}

// Every member leaves the form to the library and has one.
bool field_usable(const std::vector<fuglbm_sim *> &group) {
    return std::all_of(group.begin(), group.end(), [](fuglbm_sim *s) { return field_usable(s); });
}

// Both fused variants are the tuner's to choose from.
bool both_variants(const std::vector<fuglbm_sim *> &group, int nc, bool f32) {
    return ws_usable(nc, f32) &&
           std::all_of(group.begin(), group.end(), [](fuglbm_sim *s) { return s->auto_kernel; });
}

BatchClass batch_class(const std::vector<fuglbm_sim *> &group, int nc, bool f32) {
    int64_t strip_rows = 0;
    int ny_max = 1;
    for (auto *s : group) {
        strip_rows += (int64_t)((s->nx + FUSED_OUT - 1) / FUSED_OUT) * s->ny;
        ny_max = std::max(ny_max, s->ny);
    }
    const int tag = (both_variants(group, nc, f32) ? 0 : group[0]->kernel) +
                    (field_usable(group) ? 4 : 0);
    return {nc, (f32 ? 1 : 0) + 2 * tag, log2_class(strip_rows), log2_class(ny_max)};
}

fuglbm_status tune_batch(BatchTable &bt, const std::vector<fuglbm_sim *> &group, int nc, bool f32,
                         hipStream_t st) {
    bt.tune = Tuned{};
    if (form_fixed(group[0])) {   // and with it every member (BatchKey)
        const bool single = group[0]->form == FUGLBM_FORM_FIELDS_SINGLE;
        const int rows = group[0]->autotune
                             ? field_model_rows({group.begin(), group.end()}, single)
                             : group[0]->rows;
        fuglbm_status rc = build_batch(bt, group, st);
        if (rc == FUGLBM_OK) rc = build_field_batch(bt, group, rows, st);
        if (rc != FUGLBM_OK) return rc;
        bt.frun.single = bt.tune.single = single;
        bt.tune.frows = rows;
        bt.tune.fixed = true;
        return FUGLBM_OK;
    }
    for (auto *s : group)
        if (!s->autotune) return build_batch(bt, group, st);   // rows fixed by the caller
    const bool both = both_variants(group, nc, f32);
    int ny_max = 1;
    for (auto *s : group) ny_max = std::max(ny_max, s->ny);
    const auto key = batch_class(group, nc, f32);
    auto hit = batch_tune_cache().find(key);
    if (hit != batch_tune_cache().end()) {
        fuglbm_status rc = build_batch(bt, group, st, hit->second.rows, hit->second.kernel);
        if (rc != FUGLBM_OK) return rc;
        bt.tune = hit->second;
        bt.tune.frows = 0;   // its tables are not built (tune_batch_field)
        return FUGLBM_OK;
    }
    Tuned tn;
    float best_ms = 1e30f;
    for (int k : {2, 3}) {
        if (both ? false : k != group[0]->kernel) continue;
        if (k == 3 && !ws_usable(nc, f32)) continue;
        int r = 0;
        float ms = 0.f;
        fuglbm_status rc = time_candidates(
            tune_candidates(ny_max, 0), st, [&](int rr) { return build_batch(bt, group, st, rr, k); },
            [&]() { return launch_fused(k, nc, f32, bt.table(), 0, st); }, r,
            &ms);
        if (rc != FUGLBM_OK) return rc;
        if (ms < best_ms) {
            best_ms = ms;
            tn.kernel = k;
            tn.rows = r;
        }
    }
    tn.fused_ms = best_ms / (2 * TUNE_LAUNCHES);
    fuglbm_status rc = build_batch(bt, group, st, tn.rows, tn.kernel);
    if (rc != FUGLBM_OK) return rc;
    batch_tune_cache()[key] = bt.tune = tn;
    return FUGLBM_OK;
}

// The field form of a tuned group, timed (or answered from the cache) at its
// first run of several steps; builds its tables.
fuglbm_status tune_batch_field(BatchTable &bt, const std::vector<fuglbm_sim *> &group, int nc,
                               bool f32, hipStream_t st) {
    Tuned &c = batch_tune_cache()[batch_class(group, nc, f32)];
    if (!c.frows) {
        Tuned tn = bt.tune;
        fuglbm_status rc = time_field(
            {group.begin(), group.end()}, st,
            [&](int r, FieldRun &q) {
                fuglbm_status e = build_field_batch(bt, group, r, st);
                q = bt.frun;
                return e;
            },
            tn);
        if (rc != FUGLBM_OK) return rc;
        c = tn;
    }
    fuglbm_status rc = build_field_batch(bt, group, c.frows, st);
    if (rc != FUGLBM_OK) return rc;
    bt.frun.single = c.single;
    bt.tune = c;
    return FUGLBM_OK;
}

}  // namespace

// Batched multi-pass step (D3Q19, and D2Q9 simulations on the multi-pass
// kernels): one member table per (lattice, storage precision, tau != 1, and
// whether other members of the group take the field form), cached while the member set is the same; four launches per step over all
// members (no tuning: the multi-pass kernels have no variants), runs of
// GRAPH_STEPS steps replayed from a captured graph as for the fused tables.
struct GenBatch {
    std::vector<fuglbm_sim *> sims;
    std::vector<uint64_t> uids;
    std::vector<int> parity0;
    GenMember *dm = nullptr;
    size_t cap = 0;
    int64_t total[3] = {0, 0, 0};
    int lattice = 0, fp32 = 0, keep = 0;
    hipGraphExec_t graph = nullptr;   // GRAPH_STEPS steps starting at flip 0
    hipStream_t last_stream = nullptr;
    bool used = false;   // last_stream is meaningful
};

hipError_t gen_batch_step(const GenBatch &gb, int flip, hipStream_t st) {
    return launch_step_generic_batch(gb.lattice, gb.fp32 != 0, gb.keep != 0, gb.dm,
                                     (int)gb.sims.size(), gb.total, flip, st);
}

void drop_gen_graph(GenBatch &gb) {
    if (gb.graph) (void)hipGraphExecDestroy(gb.graph);
    gb.graph = nullptr;
}

fuglbm_status gen_batch_graph(GenBatch &gb) {
    if (gb.graph) return FUGLBM_OK;
    return capture_steps([&](int k, hipStream_t cs) { return gen_batch_step(gb, k & 1, cs); },
                         gb.graph, "multi-pass batch graph");
}

std::map<std::tuple<int, int, int, int>, GenBatch> &gen_batches() {
    static std::map<std::tuple<int, int, int, int>, GenBatch> t;
    return t;
}

fuglbm_status build_gen_batch(GenBatch &gb, const std::vector<fuglbm_sim *> &group) {
    std::vector<GenMember> m(group.size());
    int64_t acc[3] = {0, 0, 0};
    for (size_t k = 0; k < group.size(); ++k) {
        const fuglbm_sim *s = group[k];
        int64_t u[3];
        generic_units(s->lattice == FUGLBM_D2Q9 ? 0 : 1, s->N, s->nx, s->ny, s->nz, u);
        GenMember &g = m[k];
        g.c = s->dc;
        g.buf[0] = s->buf[0];
        g.buf[1] = s->buf[1];
        g.rho_f = s->rho_f;
        g.psi_f = s->psi_f;
        g.s_f = s->s_f;
        g.j_f = s->j_f;
        g.u_f = s->u_f;
        g.status = s->status;
        for (int p = 0; p < 3; ++p) g.end[p] = (acc[p] += u[p]);
        g.parity = s->parity;
        g.pad = 0;
    }
    if (acc[0] > INT32_MAX - 8 || acc[1] > INT32_MAX - 8 || acc[2] > INT32_MAX - 8)
        return fail(FUGLBM_EINVAL, "batch too large for one launch");
    if (gb.cap < m.size()) {
        if (gb.dm) HIP_TRY(hipFree(gb.dm));
        gb.dm = nullptr;
        gb.cap = 0;
        HIP_TRY(hipMalloc(&gb.dm, m.size() * sizeof(GenMember)));
        gb.cap = m.size();
    }
    HIP_TRY(hipMemcpy(gb.dm, m.data(), m.size() * sizeof(GenMember), hipMemcpyHostToDevice));
    gb.sims = group;
    gb.uids.clear();
    gb.parity0.clear();
    for (auto *s : group) {
        gb.uids.push_back(s->uid);
        gb.parity0.push_back(s->parity);
    }
    for (int p = 0; p < 3; ++p) gb.total[p] = acc[p];
    gb.lattice = group[0]->lattice == FUGLBM_D2Q9 ? 0 : 1;
    gb.fp32 = group[0]->fp32 ? 1 : 0;
    gb.keep = group[0]->hc.omega != 1.0 ? 1 : 0;
    drop_gen_graph(gb);   // captured with the old table's size
    return FUGLBM_OK;
}

// A destroyed simulation's buffers may be handed to someone else: drop every
// cached table (and its captured graph) that refers to it.
static void forget_sim_in_batches(const fuglbm_sim *s) {
    for (auto &kv : gen_batches()) {
        GenBatch &gb = kv.second;
        for (size_t k = 0; k < gb.sims.size(); ++k) {
            if (gb.sims[k] == s) {
                drop_gen_graph(gb);
                gb.sims.clear();
                gb.uids.clear();
                gb.parity0.clear();
                break;
            }
        }
    }
    for (auto &kv : batch_tables()) {
        BatchTable &bt = kv.second;
        for (size_t k = 0; k < bt.sims.size(); ++k) {
            if (bt.sims[k] == s) {
                drop_batch_graphs(bt);
                bt.sims.clear();
                bt.uids.clear();
                bt.parity0.clear();
                break;
            }
        }
    }
}

// ---- the groups of a batch ------------------------------------------------
namespace {

// A group of which some members have a field form and others do not (tau != 1,
// fixed kernel or rows) is split where the field form saves its members this
// much a step beside what it costs: the others then take a launch of their
// own, which on a small grid is all latency (64^2 x 3 5.6 us, 400 2 x 6 7.4 us
// a step).  In one table / split (us a step, one member at tau = 0.8): 512^2 x
// 10 and 64^2 x 10 115 / 48, two 512^2 x 10 202 / 137, 128^2 ... 240^2 x 3 and
// 160^2 37.8 / 29.2; left in one: two 200^2 x 5 27.2 (13.2 + 17.1), 64^2 x 3 as
// 8 + 1 14.4 (10.3 + 5.8).
constexpr double SPLIT_MS = 8e-3;

// The group's table brought up to date, on st, for a run of nsteps (tables and
// tuning); flip: the parity to step it at.
fuglbm_status prepare_batch(BatchTable &bt, const std::vector<fuglbm_sim *> &group, int nc,
                            bool f32, int64_t nsteps, hipStream_t st, int &flip) {
    // the table (and its graph) is shared state: launches queued on
    // another stream must finish before this call rebuilds or reuses it
    if (bt.used && bt.last_stream != st) HIP_TRY(hipStreamSynchronize(bt.last_stream));
    bt.last_stream = st;
    bt.used = true;
    bool same = bt.sims.size() == group.size();
    for (size_t k = 0; same && k < group.size(); ++k)
        same = bt.sims[k] == group[k] && bt.uids[k] == group[k]->uid;
    flip = 0;
    if (same) {
        flip = group[0]->parity ^ bt.parity0[0];
        for (size_t k = 0; k < group.size(); ++k)
            if ((group[k]->parity ^ bt.parity0[k]) != flip) same = false;
    }
    if (!same) {
        bt.tune = Tuned{};
        fuglbm_status rc = tune_batch(bt, group, nc, f32, st);
        if (rc != FUGLBM_OK) return rc;
        flip = 0;
    }
    // at the parities that the table was built for: the trials read the
    // current populations
    if (nsteps >= 2 && !bt.tune.fixed && !bt.tune.frows && field_usable(group) && !capturing(st)) {
        fuglbm_status rc = flip ? tune_batch(bt, group, nc, f32, st) : FUGLBM_OK;
        if (rc == FUGLBM_OK) rc = tune_batch_field(bt, group, nc, f32, st);
        if (rc != FUGLBM_OK) return rc;
        flip = 0;
    }
    return FUGLBM_OK;
}

// nsteps steps of a group on the fused kernels (its table, at parity flip).
fuglbm_status step_group(BatchTable &bt, const std::vector<fuglbm_sim *> &group, int nc, bool f32,
                         int flip, int64_t nsteps, hipStream_t st) {
    int64_t left = nsteps;
    if (field_pays(bt.tune, left)) {
        bt.frun.flip = flip;
        fuglbm_status rc = run_field(bt.frun, nc, f32, left, bt.fgraph[flip], st);
        if (rc != FUGLBM_OK) return rc;
        for (auto *s : group) {
            s->step += nsteps;
            s->taken = bt.frun.single ? FUGLBM_FORM_FIELDS_SINGLE : FUGLBM_FORM_FIELDS;
        }
        return FUGLBM_OK;
    }
    if (left >= 2 * GRAPH_STEPS && flip == 1) {
        hipError_t e = launch_fused(bt.kernel, nc, f32, bt.table(), flip, st);
        if (e != hipSuccess) return hip_fail(e, "batched step launch");
        flip = 0;
        --left;
    }
    if (left >= GRAPH_STEPS && flip == 0) {
        // replay a captured run of GRAPH_STEPS launches (even: parity returns)
        fuglbm_status rc = batch_graph(bt, nc, f32);
        if (rc != FUGLBM_OK) return rc;
        while (left >= GRAPH_STEPS) {
            HIP_TRY(hipGraphLaunch(bt.graph, st));
            left -= GRAPH_STEPS;
        }
    }
    for (; left > 0; --left) {
        hipError_t e = launch_fused(bt.kernel, nc, f32, bt.table(), flip, st);
        if (e != hipSuccess) return hip_fail(e, "batched step launch");
        flip ^= 1;
    }
    for (auto *s : group) {
        s->parity ^= (int)(nsteps & 1);
        s->step += nsteps;
        s->taken = FUGLBM_FORM_POPULATIONS;
    }
    return FUGLBM_OK;
}

// The same on the multi-pass kernels.
fuglbm_status step_gen_group(GenBatch &gb, const std::vector<fuglbm_sim *> &group, int flip,
                             int64_t nsteps, hipStream_t st) {
    int64_t left = nsteps;
    if (left >= 2 * GRAPH_STEPS && flip == 1) {
        hipError_t e = gen_batch_step(gb, flip, st);
        if (e != hipSuccess) return hip_fail(e, "batched multi-pass step launch");
        flip = 0;
        --left;
    }
    if (left >= GRAPH_STEPS && flip == 0) {
        // replay a captured run of GRAPH_STEPS steps (even: parity returns)
        fuglbm_status rc = gen_batch_graph(gb);
        if (rc != FUGLBM_OK) return rc;
        while (left >= GRAPH_STEPS) {
            HIP_TRY(hipGraphLaunch(gb.graph, st));
            left -= GRAPH_STEPS;
        }
    }
    for (; left > 0; --left) {
        hipError_t e = gen_batch_step(gb, flip, st);
        if (e != hipSuccess) return hip_fail(e, "batched multi-pass step launch");
        flip ^= 1;
    }
    for (auto *s : group) {
        s->parity ^= (int)(nsteps & 1);
        s->step += nsteps;
        s->taken = FUGLBM_FORM_POPULATIONS;
    }
    return FUGLBM_OK;
}

// Steps of a group on a stream, and about how long one takes (us).
struct GroupTask {
    double cost;
    std::function<fuglbm_status(hipStream_t)> run;
};

double group_cost(const std::vector<fuglbm_sim *> &group) {
    double c = 0.0, least = 0.0;
    for (auto *s : group) {
        const bool d3 = s->lattice == FUGLBM_D3Q19;
        c += (d3 ? 60e-6 : 15e-6) * (double)s->ns * s->N;
        least = std::max(least, d3 ? 30.0 : 8.0);
    }
    return least + c;
}

// Every task once, on st or beside it, done as far as st is concerned when st
// has done what this call enqueued on it.  The tasks go longest first to the
// lane with the least to do.
//
// A step of a small group is launch and barrier latency that leaves the chip
// idle, so groups beside each other cost little more than the longest: us a
// step at 200 steps, one after another / in lanes: 8 requests of 104^2 ...
// 240^2 and 40^3, N = 3 ... 9, FP32 storage 108 / 61; the same at 62^2 ...
// 144^2 and 24^3, FP64 85 / 45; 20 requests 254 / 185, at twice the size
// 866 / 762; 62^2 x 6 and 72^2 x 8 FP64 14.6 / 9.5.  Handing over to the
// side streams and back takes 25 to 30 us once: at one step the pair takes
// 31 / 56 us, at eight 17.3 / 17.2 us a step.  So lanes are taken where what
// they hide is estimated at twice that.
constexpr double LANE_US = 60.0;

fuglbm_status run_tasks(std::vector<GroupTask> &tasks, int64_t nsteps, hipStream_t st) {
    Lanes &L = device_stage().lanes;
    std::unique_lock<std::mutex> lock(L.use, std::defer_lock);
    double all = 0.0, longest = 0.0;
    for (auto &t : tasks) {
        all += t.cost;
        longest = std::max(longest, t.cost);
    }
    const bool side = (all - longest) * (double)nsteps >= LANE_US && !capturing(st) &&
                      lock.try_lock() && L.ready();
    if (!side) {
        for (auto &t : tasks) {
            fuglbm_status rc = t.run(st);
            if (rc != FUGLBM_OK) return rc;
        }
        return FUGLBM_OK;
    }
    std::stable_sort(tasks.begin(), tasks.end(),
                     [](const GroupTask &a, const GroupTask &b) { return a.cost > b.cost; });
    const int n = std::min<int>(LANES, (int)tasks.size());
    HIP_TRY(hipEventRecord(L.fork, st));
    for (int k = 1; k < n; ++k) HIP_TRY(hipStreamWaitEvent(L.st[k], L.fork, 0));
    double load[LANES] = {};
    fuglbm_status rc = FUGLBM_OK;
    for (auto &t : tasks) {
        const int k = (int)(std::min_element(load, load + n) - load);
        load[k] += t.cost;
        rc = t.run(k ? L.st[k] : st);
        if (rc != FUGLBM_OK) break;
    }
    // also after an error: nothing may be left running beside st
    for (int k = 1; k < n; ++k) {
        hipError_t e = hipEventRecord(L.join[k], L.st[k]);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, L.join[k], 0);
        if (e != hipSuccess) {
            (void)hipStreamSynchronize(L.st[k]);
            if (rc == FUGLBM_OK) rc = hip_fail(e, "joining a side stream");
        }
    }
    return rc;
}

}  // namespace

extern "C" fuglbm_status fuglbm_step_many(fuglbm_sim *const *sims, int32_t count, int64_t nsteps,
                                          void *hip_stream) {
    const TraceRange trace_range("fuglbm_step_many");
    if (count < 0 || (count > 0 && !sims)) return fail(FUGLBM_EINVAL, "bad sims array");
    if (nsteps < 0) return fail(FUGLBM_EINVAL, "nsteps must be >= 0");
    hipStream_t st = (hipStream_t)hip_stream;
    std::map<BatchKey, std::vector<fuglbm_sim *>> groups;
    std::vector<fuglbm_sim *> others;
    bool skipped = false;
    for (int k = 0; k < count; ++k) {
        fuglbm_sim *s = sims[k];
        if (!s) return fail(FUGLBM_EINVAL, "null sim in batch");
        for (int q = 0; q < k; ++q)
            if (sims[q] == s) return fail(FUGLBM_EINVAL, "duplicate sim in batch");
        if (s->sticky) {
            skipped = true;
            continue;
        }
        if (s->lattice == FUGLBM_D2Q9 && is_fused(s->kernel))
            groups[{s->N, s->fp32 ? 1 : 0, form_fixed(s) ? s->form : 0, 0}].push_back(s);
        else
            others.push_back(s);
    }
    for (int k = 0; k < count; ++k) {
        if (sims[k]->sticky) continue;
        fuglbm_status rc = order_after(sims[k], st);
        if (rc != FUGLBM_OK) return rc;
    }
    // what each group still needs of the host (tables, tuning) on st, and its
    // steps as a task
    std::vector<GroupTask> tasks;
    if (nsteps == 0) {   // no table either: it would be one that is not tuned
        groups.clear();
        others.clear();
    }
    std::list<std::vector<fuglbm_sim *>> parts;   // what the tasks refer to
    for (auto &kv : groups) {
        const int nc = std::get<0>(kv.first), form = std::get<2>(kv.first);
        const bool f32 = std::get<1>(kv.first) != 0;
        // a group stepped by one table; which: a split group has two more
        struct Table {
            BatchTable *bt;
            int flip;
        };
        auto prepare = [&](std::vector<fuglbm_sim *> &group, int which, Table &q) {
            q.bt = &batch_tables()[{nc, f32 ? 1 : 0, form, which}];
            return prepare_batch(*q.bt, group, nc, f32, nsteps, st, q.flip);
        };
        auto task = [&](std::vector<fuglbm_sim *> &group, Table q) {
            tasks.push_back({group_cost(group), [q, &group, nc, f32, nsteps](hipStream_t to) {
                                 return step_group(*q.bt, group, nc, f32, q.flip, nsteps, to);
                             }});
        };
        // members with a field form beside others without (tau != 1, fixed
        // kernel or rows)
        std::vector<fuglbm_sim *> &fields = parts.emplace_back(), &rest = parts.emplace_back();
        for (auto *s : kv.second) (field_usable(s) ? fields : rest).push_back(s);
        Table q{}, p{};
        if (nsteps >= 2 && !fields.empty() && !rest.empty() && !capturing(st)) {
            fuglbm_status rc = prepare(fields, 1, q);
            if (rc != FUGLBM_OK) return rc;
            if (field_pays(q.bt->tune, nsteps, SPLIT_MS)) {
                rc = prepare(rest, 2, p);
                if (rc != FUGLBM_OK) return rc;
                task(fields, q);
                task(rest, p);
                continue;
            }
        }
        fuglbm_status rc = prepare(kv.second, 0, q);
        if (rc != FUGLBM_OK) return rc;
        task(kv.second, q);
    }
    // multi-pass members by (lattice, precision, tau != 1): those that take the
    // field form do so one by one, the others share one table
    std::map<std::tuple<int, int, int>, std::vector<fuglbm_sim *>> ggroups;
    for (auto *s : others)
        ggroups[{s->lattice, s->fp32 ? 1 : 0, s->hc.omega != 1.0 ? 1 : 0}].push_back(s);
    for (auto &kv : ggroups) {
        std::vector<fuglbm_sim *> &fields = parts.emplace_back(), &group = parts.emplace_back();
        split_forms3(kv.second, nsteps, fields, group);
        if (!fields.empty())
            tasks.push_back({group_cost(fields), [&fields, nsteps](hipStream_t to) {
                                 for (auto *s : fields) {
                                     fuglbm_status rc = run_field3(s, nsteps, to);
                                     if (rc != FUGLBM_OK) return rc;
                                 }
                                 return FUGLBM_OK;
                             }});
        if (group.empty()) continue;
        GenBatch &gb = gen_batches()[std::tuple_cat(kv.first, std::make_tuple(fields.empty() ? 0 : 1))];
        // the table is shared state: launches queued on another stream must
        // finish before this call rebuilds or reuses it
        if (gb.used && gb.last_stream != st) HIP_TRY(hipStreamSynchronize(gb.last_stream));
        gb.last_stream = st;
        gb.used = true;
        bool same = gb.sims.size() == group.size();
        for (size_t k = 0; same && k < group.size(); ++k)
            same = gb.sims[k] == group[k] && gb.uids[k] == group[k]->uid;
        int flip = 0;
        if (same) {
            flip = group[0]->parity ^ gb.parity0[0];
            for (size_t k = 0; k < group.size(); ++k)
                if ((group[k]->parity ^ gb.parity0[k]) != flip) same = false;
        }
        if (!same) {
            // launches queued on st may still read the table that the
            // rebuild overwrites (the upload is not ordered after them)
            HIP_TRY(hipStreamSynchronize(st));
            fuglbm_status rc = build_gen_batch(gb, group);
            if (rc != FUGLBM_OK) return rc;
            flip = 0;
        }
        tasks.push_back({group_cost(group), [&gb, &group, flip, nsteps](hipStream_t to) {
                             return step_gen_group(gb, group, flip, nsteps, to);
                         }});
    }
    {
        fuglbm_status rc = run_tasks(tasks, nsteps, st);
        if (rc != FUGLBM_OK) return rc;
    }
    for (int k = 0; k < count; ++k) {
        if (sims[k]->sticky) continue;
        fuglbm_status rc = mark_done(sims[k], st);
        if (rc != FUGLBM_OK) return rc;
    }
    if (skipped) return fail(FUGLBM_ENONFINITE, "some simulations have a sticky device error");
    return FUGLBM_OK;
}

// ---------------------------------------------------------------------------
// Batched stepping without allocation (fuglbm_step_many_noalloc).
//
// The batch's work tables (per-member pointers and geometry, then the work
// items in the same XCD-dealt order as fuglbm_step_many) live in `scratch`,
// a file-scope device array of fixed size that every call on a device
// shares.  They are written on the device by a table kernel whose member
// data arrive as kernel arguments, so a call needs no device allocation,
// no graph instantiation and no copy from host memory; the steps are plain
// launches of the fused kernel.  `scratch` is a host-side stand-in in host
// code: its device address is looked up once per device
// (hipGetSymbolAddress) and only that address is ever passed on.
// ---------------------------------------------------------------------------
namespace {

constexpr int NA_MAX_MEMBERS = 256;                // simulations per call
constexpr int NA_MAX_ITEMS = 65536;                // fused work items per call
constexpr int NA_CHUNK = 32;                       // members per table-kernel launch
constexpr size_t NA_GEOM_OFF = 0;                  // int4 {nx, ny, rows, first item}
constexpr size_t NA_SIMS_OFF = NA_GEOM_OFF + 16 * NA_MAX_MEMBERS;
constexpr size_t NA_ITEMS_OFF = NA_SIMS_OFF + sizeof(FusedSim) * NA_MAX_MEMBERS;
constexpr size_t NA_SCRATCH_BYTES = NA_ITEMS_OFF + sizeof(FusedItem) * NA_MAX_ITEMS;

static __device__ __align__(256) unsigned char scratch[NA_SCRATCH_BYTES];

struct NaMember {
    const SimConst *c;
    void *buf0, *buf1;
    uint32_t *status;
    int32_t parity, nx, ny, rows;
};

struct NaChunk {
    int32_t base;                 // index of m[0] among the group's members
    int32_t count;                // members in this chunk
    int32_t first[NA_CHUNK];      // each member's first logical item in the group
    NaMember m[NA_CHUNK];
};

// Members [base, base + count) of one group: pointers and geometry.
__global__ void k_na_members(NaChunk a, FusedSim *sims, int4 *geom) {
    const int t = threadIdx.x;
    if (t >= a.count) return;
    const NaMember &m = a.m[t];
    FusedSim fs;
    fs.c = m.c;
    fs.buf[0] = m.buf0;
    fs.buf[1] = m.buf1;
    fs.status = m.status;
    fs.parity = m.parity;
    fs.nx = m.nx;
    fs.ny = m.ny;
    fs.pad = 0;
    sims[a.base + t] = fs;
    geom[a.base + t] = make_int4(m.nx, m.ny, m.rows, a.first[t]);
}

// Work items of one group: logical item li (member-major, then chunk of
// rows, then strip) goes to slot (li % per) * 8 + li / per, so XCD k
// (workgroups are dealt round-robin) runs the k-th contiguous slice.
__global__ void k_na_items(const int4 *geom, int nmem, int nlogical, int per, FusedItem *items) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= per * 8) return;
    const int li = (b % 8) * per + b / 8;
    FusedItem it{-1, 0, 0, 0};
    if (li < nlogical) {
        int k = 0;
        while (k + 1 < nmem && geom[k + 1].w <= li) ++k;
        const int4 g = geom[k];
        const int strips = (g.x + FUSED_OUT - 1) / FUSED_OUT;
        const int local = li - g.w;
        const int c = local / strips, t = local % strips;
        it.sim = k;
        it.x0 = t * FUSED_OUT;
        it.y0 = c * g.z;
        it.rows = min(g.z, g.y - c * g.z);
    }
    items[b] = it;
}

std::mutex na_mutex;
void *na_ptr[64];

// Device address of `scratch` on the current device (looked up once).
fuglbm_status na_scratch(char **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(FUGLBM_EDEVICE, "device index out of range");
    std::lock_guard<std::mutex> lk(na_mutex);
    if (!na_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        na_ptr[dev] = p;
    }
    *out = (char *)na_ptr[dev];
    return FUGLBM_OK;
}

}  // namespace

extern "C" fuglbm_status fuglbm_step_many_noalloc(fuglbm_sim *const *sims, int32_t count,
                                                  int64_t nsteps, void *hip_stream) {
    const TraceRange trace_range("fuglbm_step_many_noalloc");
    if (count < 0 || (count > 0 && !sims)) return fail(FUGLBM_EINVAL, "bad sims array");
    if (nsteps < 0) return fail(FUGLBM_EINVAL, "nsteps must be >= 0");
    if (count > NA_MAX_MEMBERS)
        return fail(FUGLBM_EINVAL, "at most 256 simulations per call");
    hipStream_t st = (hipStream_t)hip_stream;
    // members by (ncomp, precision) class, in call order; sticky ones skipped
    int cls[NA_MAX_MEMBERS];
    int key[NA_MAX_MEMBERS], nkeys = 0;
    bool skipped = false;
    int64_t total_items = 0;
    for (int k = 0; k < count; ++k) {
        fuglbm_sim *s = sims[k];
        if (!s) return fail(FUGLBM_EINVAL, "null sim in batch");
        for (int q = 0; q < k; ++q)
            if (sims[q] == s) return fail(FUGLBM_EINVAL, "duplicate sim in batch");
        if (s->lattice != FUGLBM_D2Q9 || !is_fused(s->kernel))
            return fail(FUGLBM_EINVAL, "only D2Q9 simulations on a fused kernel");
        if (s->rows < 1) return fail(FUGLBM_EINVAL, "simulation without fused rows");
        cls[k] = -1;
        if (s->sticky) {
            skipped = true;
            continue;
        }
        const int kk = s->N * 2 + (s->fp32 ? 1 : 0);
        int g = 0;
        while (g < nkeys && key[g] != kk) ++g;
        if (g == nkeys) key[nkeys++] = kk;
        cls[k] = g;
        const int64_t strips = (s->nx + FUSED_OUT - 1) / FUSED_OUT;
        total_items += strips * ((s->ny + s->rows - 1) / s->rows) + 7;   // + XCD padding
    }
    if (total_items > NA_MAX_ITEMS)
        return fail(FUGLBM_EINVAL, "batch needs more than 65536 work items");
    if (nkeys == 0 || nsteps == 0) {
        if (skipped) return fail(FUGLBM_ENONFINITE, "some simulations have a sticky device error");
        return FUGLBM_OK;
    }
    char *base = nullptr;
    fuglbm_status rc = na_scratch(&base);
    if (rc != FUGLBM_OK) return rc;
    int4 *geom = (int4 *)(base + NA_GEOM_OFF);
    FusedSim *dsims = (FusedSim *)(base + NA_SIMS_OFF);
    FusedItem *ditems = (FusedItem *)(base + NA_ITEMS_OFF);
    int mem_off = 0, item_off = 0;
    for (int g = 0; g < nkeys; ++g) {
        // this group's members, their first logical items
        NaChunk ch;
        int nmem = 0, nlogical = 0;
        fuglbm_sim *first = nullptr;
        ch.base = 0;
        ch.count = 0;
        for (int k = 0; k < count; ++k) {
            if (cls[k] != g) continue;
            fuglbm_sim *s = sims[k];
            if (!first) first = s;
            NaMember &m = ch.m[ch.count];
            m.c = s->dc;
            m.buf0 = s->buf[0];
            m.buf1 = s->buf[1];
            m.status = s->status;
            m.parity = s->parity;
            m.nx = s->nx;
            m.ny = s->ny;
            m.rows = s->rows;
            ch.first[ch.count] = nlogical;
            nlogical += ((s->nx + FUSED_OUT - 1) / FUSED_OUT) * ((s->ny + s->rows - 1) / s->rows);
            ++ch.count;
            ++nmem;
            if (ch.count == NA_CHUNK) {
                hipLaunchKernelGGL(k_na_members, dim3(1), dim3(NA_CHUNK), 0, st, ch,
                                   dsims + mem_off, geom + mem_off);
                ch.base += NA_CHUNK;
                ch.count = 0;
            }
        }
        if (ch.count > 0)
            hipLaunchKernelGGL(k_na_members, dim3(1), dim3(NA_CHUNK), 0, st, ch, dsims + mem_off,
                               geom + mem_off);
        const int per = (nlogical + 7) / 8;
        const int nitems = per * 8;
        hipLaunchKernelGGL(k_na_items, dim3((nitems + 255) / 256), dim3(256), 0, st,
                           geom + mem_off, nmem, nlogical, per, ditems + item_off);
        HIP_TRY(hipGetLastError());
        const int ncomp = first->N;
        const bool f32 = first->fp32;
        const int kern = first->kernel == 3 && ws_usable(ncomp, f32) ? 3 : 2;
        int rows = 0;
        for (int k = 0; k < count; ++k)
            if (cls[k] == g) rows = std::max(rows, sims[k]->rows);
        for (int64_t t = 0; t < nsteps; ++t) {
            const FusedTable tab{ditems + item_off, nitems, dsims + mem_off, nmem, rows};
            hipError_t e = launch_fused(kern, ncomp, f32, tab, (int)(t & 1), st);
            if (e != hipSuccess) return hip_fail(e, "batched step launch");
        }
        mem_off += nmem;
        item_off += nitems;
    }
    for (int k = 0; k < count; ++k) {
        if (cls[k] < 0) continue;
        fuglbm_sim *s = sims[k];
        s->parity ^= (int)(nsteps & 1);
        s->step += nsteps;
        if (nsteps) s->taken = FUGLBM_FORM_POPULATIONS;
        s->last_stream = st;
        s->done_valid = false;   // not recorded here (the caller orders streams)
    }
    if (skipped) return fail(FUGLBM_ENONFINITE, "some simulations have a sticky device error");
    return FUGLBM_OK;
}
