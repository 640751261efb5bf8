// HeteroConv layer: per-graph context and the forward / backward schedules.  The three relation modules (near, pins,
// pinned) are independent of one another up to the merge at the cells (paper Section 3.4: independent sub-graph updates
// launched together).  A step of the layer is ONE launch in which the workgroups of all relations -- and, in a model, of
// all sub-graphs -- run side by side: a forward is three launches (D-ReLU, DR-SpMM, projections), a backward two or three (weight
// gradients beside projection gradients; transposed DR-SpMM of a placed `near` on staged tiles; the other transposed DR-SpMMs with the
// dense input gradients, and the sums over the weight gradients' partials behind them).  Three streams joined by events did the
// same with 24 launches and some 30 event operations; a 2048-cell layer pass then took 0.21 ms, nearly all of it launch and event
// overhead; with five launches backward 0.067 ms, now 0.050.
// Everything runs on the caller's stream, in order; the host does not wait inside fwd / bwd, except in the first backward pass
// of a context that is called on another stream than the one before it (the scratch is the context's).
#include "dr_internal.h"

#include <new>
#include <vector>

namespace {
// kernel ids for the optional per-kernel timing (heteroconv_profile / heteroconv_kernel_times)
enum KernelId {
    kTopkCell, kTopkNet, kFwdNear, kFwdPins, kFwdPinned, kProjCell, kProjPins,
    kWgCell, kWgPins, kDhCell, kDhPins, kBwdNear, kBwdNearPins, kBwdPins, kBwdPinned, kNumKernels
};
const char* const kKernelNames[kNumKernels] = {
    "dr_topk.cell", "dr_topk.net", "dr_spmm_fwd.near", "dr_spmm_fwd.pins", "dr_spmm_fwd.pinned",
    "proj.cell+merge", "proj.pins", "wgrad.cell", "wgrad.pins", "dproj.cell", "dproj.pins",
    "dr_spmm_bwd.near", "dr_spmm_bwd.near+pins+dX", "dr_spmm_bwd.pins+dX", "dr_spmm_bwd.pinned+dX"};
struct TimedLaunch { int id; hipEvent_t start, stop; bool start_shared; };   // start_shared: start is the previous launch's stop
}  // namespace

struct dr_heteroconv {
    int64_t Nc, Nn;
    int D;
    // D-ReLU widths: k_near (cells, source and self term of near), k_pins (cells, source of pins), k_self (nets,
    // self term of pins), k_pinned (nets, source of pinned).  Equal widths on one node type share one CBSR.
    int k_near, k_pins, k_self, k_pinned;
    dr_csr A[3];        // near, pins, pinned (borrowed)
    dr_csr At[3];       // transposes (owned)
    // what the owned buffers were sized for; a context can be re-bound to any graph within these bounds
    int64_t cap_Nc, cap_Nn, cap_E[3];
    int32_t* t_rp[3];   // buffers behind At[]
    int32_t* t_ci[3];
    float* t_v[3];
    void* t_ws[3];      // transpose workspaces (kept only by re-bindable contexts)
    size_t t_wsb[3];
    void* owned[32];
    int n_owned;
    // backward scratch
    float* dH;          // [Nc,D] near | [Nn,D] pins, behind one another so that one kernel can gather both
    float* dH_pinned;   // [Nc,D]
    float* S_cell;      // [Nc,k_near]  near self-term gradient at the near selection (plus near's own piece, where that is summed apart)
    float* S_net;       // [Nn,k_self]  pins self-term gradient at its selection
    float* G_pins;      // [Nc,k_pins]   pins piece, only where it needs a buffer of its own
    float* G_pinned;    // [Nn,k_pinned] pinned piece, likewise
    void* wg_scratch[2];   // cells, nets
    drc::PartialSum* wg_sums;   // [kMaxGraphs * kSumsPerGraph] the sums over that scratch that a pass of several graphs leaves to a later launch
    // The scratch above is one for all backward passes of a context: a pass on another stream than the last one's waits for it.
    // The first change of streams waits on the host; from then on every pass records `end`, and a change waits on the device.
    // (A context that stays on one stream does without the event: it is a packet of its own for the GPU, 3 us of a 70 us layer.
    // Recording it later, when the stream changes, would use a stream that its owner may have destroyed since.)
    hipStream_t last_stream;
    bool has_last, many_streams, end_recorded;
    hipEvent_t end;
    int device;
    int overlap;        // DR_OVERLAP_*: whether the relations of a step share a launch
    dr_spmm_plan* near_plan;   // transposed `near` with its dH rows staged in LDS tile by tile (heteroconv_set_cell_order), or null
    // optional per-kernel timing
    bool profile;
    std::vector<TimedLaunch>* timed;      // launches recorded since the last heteroconv_kernel_times
    std::vector<hipEvent_t>* event_pool;  // idle timing events
    hipEvent_t chain_stop;                // stop event of the previous timed launch of this call: the start of the next one
};

using namespace drc;

// Staging the gathered rows of a tile pays from about two edges per staged row on (measured on the 1.2 M-cell `near`
// relation: 0.64 ms at 2.1, 0.42 ms at 4.7, against 0.67 ms for the plain gather).
static constexpr double kMinStagingReuse = 2.0;

// Whether the launch that writes dX sums the transposed `near` sooner than a launch of its own on staged tiles, which every step has to
// wait for: beside pins (one cell width), while wavefronts of 8 rows fit the chip at once (kSmallLaunch).  Backward of 2 048 / 10 000 /
// 20 000 cells, D = 64, staged / beside pins: 33 / 29, 49 / 44, 60 / 52 us; 33 000: 81 / 87.
static bool near_beside_pins(const dr_heteroconv* c) {
    return c->k_pins == c->k_near && c->k_near <= kDenseMaxK && c->Nc + c->Nn <= kSmallLaunch;
}

HeteroDims drc::heteroconv_dims(const dr_heteroconv* c) {
    return HeteroDims{c->Nc, c->Nn, c->D, c->k_near, c->k_pins, c->k_self, c->k_pinned};
}

namespace {

int dev_alloc(dr_heteroconv* c, void** p, size_t bytes) {
    *p = nullptr;
    bytes += 1024;                        // a gather may read row 0 of an empty array
    DRC_HIP(hipMalloc(p, bytes));
    c->owned[c->n_owned++] = *p;
    return DR_OK;
}

void release(dr_heteroconv* c) {
    if (!c) return;
    spmm_plan_destroy(c->near_plan);
    if (c->end) (void)hipEventDestroy(c->end);
    for (int i = 0; i < c->n_owned; ++i) (void)hipFree(c->owned[i]);
    if (c->timed) {
        for (TimedLaunch& t : *c->timed) { if (!t.start_shared) (void)hipEventDestroy(t.start); (void)hipEventDestroy(t.stop); }
        delete c->timed;
    }
    if (c->event_pool) {
        for (hipEvent_t e : *c->event_pool) (void)hipEventDestroy(e);
        delete c->event_pool;
    }
    delete c;
}

// Brackets one launch with timing events when profiling is on.  The launches of a call run back to back on one stream, so
// the stop event of one launch also serves as the start of the next: one event record per launch instead of two (each
// record is a packet the GPU has to process).
struct ScopedTiming {
    dr_heteroconv* c; hipStream_t s; TimedLaunch t; bool on;
    hipEvent_t take() {
        hipEvent_t e = nullptr;
        if (!c->event_pool->empty()) { e = c->event_pool->back(); c->event_pool->pop_back(); }
        else if (hipEventCreate(&e) != hipSuccess) e = nullptr;
        return e;
    }
    ScopedTiming(dr_heteroconv* c_, int id, hipStream_t s_) : c(c_), s(s_), t{id, nullptr, nullptr, false}, on(false) {
        if (!c->profile) return;
        if (c->chain_stop) {
            t.start = c->chain_stop;
            t.start_shared = true;
            t.stop = take();
            on = t.stop != nullptr;
        } else {
            t.start = take();
            t.stop = take();
            if (t.start && t.stop && hipEventRecord(t.start, s) == hipSuccess) on = true;
        }
    }
    ~ScopedTiming() {
        if (!on) return;
        (void)hipEventRecord(t.stop, s);
        c->timed->push_back(t);
        c->chain_stop = t.stop;
    }
};

}  // namespace

const dr_csr* drc::heteroconv_relations(const dr_heteroconv* c) { return c->A; }

void drc::heteroconv_capacity(const dr_heteroconv* c, int64_t* cells, int64_t* nets) { *cells = c->cap_Nc; *nets = c->cap_Nn; }

static int check_widths(int32_t D, int32_t k_near, int32_t k_pins, int32_t k_self, int32_t k_pinned) {
    DRC_REQUIRE(k_near >= 1 && k_pins >= 1 && k_self >= 1 && k_pinned >= 1, "heteroconv_create: k must be >= 1");
    DRC_REQUIRE(k_near <= D && k_pins <= D && k_self <= D && k_pinned <= D, "heteroconv_create: k exceeds D");
    if (!(D == 32 || D == 64 || D == 96 || D == 128))
        return fail(DR_ERR_UNSUPPORTED, "heteroconv_create: D = %d not in {32,64,96,128}", D);
    return DR_OK;
}

int drc::heteroconv_create_capacity(dr_heteroconv** ctx, int64_t Nc, int64_t Nn, const int64_t E[3], int32_t D, int32_t k_near,
                                    int32_t k_pins, int32_t k_self, int32_t k_pinned, bool keep_workspace) {
    DRC_REQUIRE(ctx != nullptr, "heteroconv_create: null ctx");
    *ctx = nullptr;
    DRC_TRY(check_widths(D, k_near, k_pins, k_self, k_pinned));
    DRC_REQUIRE(Nc >= 0 && Nn >= 0 && E[0] >= 0 && E[1] >= 0 && E[2] >= 0, "heteroconv_create: negative size");
    DRC_REQUIRE(E[0] < (int64_t(1) << 31) && E[1] < (int64_t(1) << 31) && E[2] < (int64_t(1) << 31), "heteroconv_create: nnz >= 2^31");
    DRC_REQUIRE(Nc * (int64_t)D < (int64_t(1) << 31) * 2 && Nn * (int64_t)D < (int64_t(1) << 31) * 2,
                "heteroconv_create: n*D too large");

    dr_heteroconv* c = new (std::nothrow) dr_heteroconv();
    DRC_REQUIRE(c != nullptr, "heteroconv_create: out of host memory");
    c->Nc = Nc; c->Nn = Nn; c->D = D;
    c->cap_Nc = Nc; c->cap_Nn = Nn;
    for (int i = 0; i < 3; ++i) c->cap_E[i] = E[i];
    c->k_near = k_near; c->k_pins = k_pins; c->k_self = k_self; c->k_pinned = k_pinned;
    c->timed = new (std::nothrow) std::vector<TimedLaunch>();
    c->event_pool = new (std::nothrow) std::vector<hipEvent_t>();

    int rc = DR_OK;
    auto bail = [&](int code) { release(c); return code; };
    if (hipEventCreateWithFlags(&c->end, hipEventDisableTiming) != hipSuccess) return bail(hip_fail(hipGetLastError(), "hipEventCreate"));
    if (hipGetDevice(&c->device) != hipSuccess) return bail(hip_fail(hipGetLastError(), "hipGetDevice"));

    // buffers of the transposed adjacencies: A^T of relation i has as many rows as A has columns
    const int64_t t_rows[3] = {Nc, Nc, Nn}, a_rows[3] = {Nc, Nn, Nc};
    for (int i = 0; i < 3; ++i) {
        if ((rc = dev_alloc(c, (void**)&c->t_rp[i], 4 * (size_t)(t_rows[i] + 1)))) return bail(rc);
        if ((rc = dev_alloc(c, (void**)&c->t_ci[i], 4 * (size_t)E[i]))) return bail(rc);
        if ((rc = dev_alloc(c, (void**)&c->t_v[i], 4 * (size_t)E[i]))) return bail(rc);
        c->t_wsb[i] = dr_csr_transpose_workspace_bytes(a_rows[i], t_rows[i], E[i]);
        if (keep_workspace && (rc = dev_alloc(c, &c->t_ws[i], c->t_wsb[i]))) return bail(rc);
    }
    if ((rc = dev_alloc(c, (void**)&c->dH, 4 * (size_t)(Nc + Nn) * D))) return bail(rc);
    if ((rc = dev_alloc(c, (void**)&c->dH_pinned, 4 * (size_t)Nc * D))) return bail(rc);
    if ((rc = dev_alloc(c, &c->wg_scratch[0], wgrad_scratch_bytes(Nc, D, 3)))) return bail(rc);
    if ((rc = dev_alloc(c, &c->wg_scratch[1], wgrad_scratch_bytes(Nn, D, 2)))) return bail(rc);
    if ((rc = dev_alloc(c, (void**)&c->wg_sums, sizeof(PartialSum) * kMaxGraphs * kSumsPerGraph))) return bail(rc);
    if ((rc = dev_alloc(c, (void**)&c->S_cell, 4 * (size_t)Nc * k_near))) return bail(rc);
    if ((rc = dev_alloc(c, (void**)&c->S_net, 4 * (size_t)Nn * k_self))) return bail(rc);
    if (k_pins != k_near && k_pins > kDenseMaxK && (rc = dev_alloc(c, (void**)&c->G_pins, 4 * (size_t)Nc * k_pins))) return bail(rc);
    if (k_self != k_pinned && k_pinned > kDenseMaxK && (rc = dev_alloc(c, (void**)&c->G_pinned, 4 * (size_t)Nn * k_pinned))) return bail(rc);
    *ctx = c;
    return DR_OK;
}

// Binds three relations (device CSRs within the context's capacity) and enqueues their transposition on `s`.
// Nothing here waits for the device; work enqueued on the context after `s` has passed this point sees the new graph.
int drc::heteroconv_bind(dr_heteroconv* c, const dr_csr* near, const dr_csr* pins, const dr_csr* pinned, hipStream_t s) {
    if (int rc = check_csr(near, "heteroconv_bind: near", true)) return rc;
    if (int rc = check_csr(pins, "heteroconv_bind: pins", true)) return rc;
    if (int rc = check_csr(pinned, "heteroconv_bind: pinned", true)) return rc;
    DRC_REQUIRE(near->n_rows == near->n_cols, "heteroconv_bind: near must be square (cell x cell)");
    const int64_t Nc = near->n_rows, Nn = pins->n_rows;
    DRC_REQUIRE(pins->n_cols == Nc, "heteroconv_bind: pins must be Nn x Nc");
    DRC_REQUIRE(pinned->n_rows == Nc && pinned->n_cols == Nn, "heteroconv_bind: pinned must be Nc x Nn");
    DRC_REQUIRE(Nc <= c->cap_Nc && Nn <= c->cap_Nn && near->nnz <= c->cap_E[0] && pins->nnz <= c->cap_E[1] &&
                    pinned->nnz <= c->cap_E[2],
                "heteroconv_bind: graph (%lld cells, %lld nets, %lld / %lld / %lld edges) exceeds the context's capacity",
                (long long)Nc, (long long)Nn, (long long)near->nnz, (long long)pins->nnz, (long long)pinned->nnz);
    c->Nc = Nc; c->Nn = Nn;
    c->A[0] = *near; c->A[1] = *pins; c->A[2] = *pinned;
    if (c->near_plan) {      // made for the graph bound before
        DRC_HIP(hipDeviceSynchronize());
        spmm_plan_destroy(c->near_plan);
        c->near_plan = nullptr;
    }
    TransposeJob jobs[3];
    for (int i = 0; i < 3; ++i) {
        const dr_csr& A = c->A[i];
        DRC_REQUIRE(c->t_ws[i] != nullptr, "heteroconv_bind: context without transpose workspace");
        jobs[i] = TransposeJob{&c->A[i], c->t_rp[i], c->t_ci[i], c->t_v[i], c->t_ws[i]};
        c->At[i] = dr_csr{A.n_cols, A.n_rows, A.nnz, c->t_rp[i], c->t_ci[i], c->t_v[i]};
    }
    DRC_TRY(launch_csr_transposes(jobs, 3, s));
    return DR_OK;
}

int drc::heteroconv_create_widths(dr_heteroconv** ctx, const dr_csr* near, const dr_csr* pins, const dr_csr* pinned, int32_t D,
                                  int32_t k_near, int32_t k_pins, int32_t k_self, int32_t k_pinned) {
    DRC_REQUIRE(ctx != nullptr, "heteroconv_create: null ctx");
    *ctx = nullptr;
    if (int rc = check_csr(near, "heteroconv_create: near", true)) return rc;
    if (int rc = check_csr(pins, "heteroconv_create: pins", true)) return rc;
    if (int rc = check_csr(pinned, "heteroconv_create: pinned", true)) return rc;
    DRC_REQUIRE(near->n_rows == near->n_cols, "heteroconv_create: near must be square (cell x cell)");
    const int64_t Nc = near->n_rows, Nn = pins->n_rows;
    DRC_REQUIRE(pins->n_cols == Nc, "heteroconv_create: pins must be Nn x Nc");
    DRC_REQUIRE(pinned->n_rows == Nc && pinned->n_cols == Nn, "heteroconv_create: pinned must be Nc x Nn");
    DRC_TRY(check_widths(D, k_near, k_pins, k_self, k_pinned));
    // the caller may still be producing the CSR arrays on another stream
    DRC_HIP(hipDeviceSynchronize());
    const int64_t E[3] = {near->nnz, pins->nnz, pinned->nnz};
    dr_heteroconv* c = nullptr;
    DRC_TRY(heteroconv_create_capacity(&c, Nc, Nn, E, D, k_near, k_pins, k_self, k_pinned, false));
    // one-off transposition: the workspaces are released again
    int rc = DR_OK;
    for (int i = 0; i < 3 && rc == DR_OK; ++i)
        if (hipMalloc(&c->t_ws[i], c->t_wsb[i] ? c->t_wsb[i] : 256) != hipSuccess) rc = hip_fail(hipGetLastError(), "hipMalloc(transpose workspace)");
    if (rc == DR_OK) rc = heteroconv_bind(c, near, pins, pinned, nullptr);
    const hipError_t e = hipDeviceSynchronize();
    for (int i = 0; i < 3; ++i) {
        if (c->t_ws[i]) (void)hipFree(c->t_ws[i]);
        c->t_ws[i] = nullptr;
    }
    if (rc == DR_OK && e != hipSuccess) rc = hip_fail(e, "hipDeviceSynchronize(transpose)");
    if (rc != DR_OK) { release(c); return rc; }
    *ctx = c;
    return DR_OK;
}

extern "C" {

int heteroconv_create(dr_heteroconv** ctx, const dr_csr* near, const dr_csr* pins, const dr_csr* pinned,
                      int32_t D, int32_t k_cell, int32_t k_net) {
    return heteroconv_create_widths(ctx, near, pins, pinned, D, k_cell, k_cell, k_net, k_net);
}

int heteroconv_create_per_relation(dr_heteroconv** ctx, const dr_csr* near, const dr_csr* pins, const dr_csr* pinned,
                                   int32_t D, int32_t k_near, int32_t k_pins, int32_t k_pinned) {
    return heteroconv_create_widths(ctx, near, pins, pinned, D, k_near, k_pins, k_pins, k_pinned);
}

int heteroconv_get_k(const dr_heteroconv* ctx, int32_t* k_near, int32_t* k_pins, int32_t* k_self, int32_t* k_pinned) {
    DRC_REQUIRE(ctx && k_near && k_pins && k_self && k_pinned, "heteroconv_get_k: null argument");
    *k_near = ctx->k_near; *k_pins = ctx->k_pins; *k_self = ctx->k_self; *k_pinned = ctx->k_pinned;
    return DR_OK;
}

int heteroconv_destroy(dr_heteroconv* ctx) {
    if (!ctx) return DR_OK;
    (void)hipDeviceSynchronize();
    release(ctx);
    return DR_OK;
}

int heteroconv_get_transpose(const dr_heteroconv* ctx, int which, dr_csr* out) {
    DRC_REQUIRE(ctx && out, "heteroconv_get_transpose: null argument");
    DRC_REQUIRE(which >= 0 && which < 3, "heteroconv_get_transpose: which must be 0, 1 or 2");
    *out = ctx->At[which];
    return DR_OK;
}

int heteroconv_set_cell_order(dr_heteroconv* ctx, const int32_t* cell_order, int* staged, void* stream) {
    DRC_REQUIRE(ctx != nullptr, "heteroconv_set_cell_order: null context");
    if (staged) *staged = 0;
    if (ctx->near_plan) {
        DRC_HIP(hipDeviceSynchronize());      // work that still reads the old plan
        spmm_plan_destroy(ctx->near_plan);
        ctx->near_plan = nullptr;
    }
    if (ctx->At[0].nnz == 0) return DR_OK;
    const int cw = ctx->D % 64 == 0 ? 64 : 32;
    if (ctx->D % 32 != 0 || ctx->D / cw > 4 || ctx->k_near > 2 * cw) return DR_OK;      // widths the staged kernel does not cover
    dr_spmm_plan* plan = nullptr;
    const int rc = spmm_plan_create(&plan, &ctx->At[0], cell_order, ctx->D, as_stream(stream));
    if (rc == DR_ERR_UNSUPPORTED) return DR_OK;        // a row that does not fit a tile: the plain kernel stays
    if (rc != DR_OK) return rc;
    int64_t n_tiles = 0;
    double reuse = 0.0;
    DRC_TRY(dr_spmm_plan_info(plan, &n_tiles, &reuse));
    // Nothing to gain from staging: rows of a tile share too few neighbours, or the graph is small.  (The plan was made all the same: it
    // is what refuses an order that is no permutation.)
    if (reuse < kMinStagingReuse || near_beside_pins(ctx)) {
        spmm_plan_destroy(plan);
        return DR_OK;
    }
    ctx->near_plan = plan;
    if (staged) *staged = 1;
    return DR_OK;
}

int heteroconv_set_overlap(dr_heteroconv* ctx, int mode) {
    DRC_REQUIRE(ctx != nullptr, "heteroconv_set_overlap: null context");
    DRC_REQUIRE(mode == DR_OVERLAP_AUTO || mode == DR_OVERLAP_ON || mode == DR_OVERLAP_OFF,
                "heteroconv_set_overlap: unknown mode %d", mode);
    ctx->overlap = mode;
    return DR_OK;
}

int heteroconv_profile(dr_heteroconv* ctx, int enable) {
    DRC_REQUIRE(ctx != nullptr, "heteroconv_profile: null context");
    DRC_REQUIRE(ctx->timed && ctx->event_pool, "heteroconv_profile: out of host memory");
    ctx->profile = enable != 0;
    return DR_OK;
}

int heteroconv_profile_k(dr_heteroconv* c, const float* X_cell, const float* X_net, const int32_t* candidates,
                         int32_t n_candidates, int32_t warmup, int32_t reps, float* ms_fwd, float* ms_bwd,
                         int32_t* best_k) {
    DRC_REQUIRE(c != nullptr, "heteroconv_profile_k: null context");
    DRC_REQUIRE(X_cell && X_net && candidates && ms_fwd && ms_bwd && best_k, "heteroconv_profile_k: null argument");
    DRC_REQUIRE(aligned(X_cell, 16) && aligned(X_net, 16), "heteroconv_profile_k: embeddings must be 16-byte aligned");
    DRC_REQUIRE(n_candidates >= 1 && n_candidates <= 64, "heteroconv_profile_k: n_candidates = %d out of range [1, 64]", n_candidates);
    DRC_REQUIRE(warmup >= 0 && reps >= 1 && reps <= 1000, "heteroconv_profile_k: warmup = %d, reps = %d", warmup, reps);
    int kmax = 0;
    for (int i = 0; i < n_candidates; ++i) {
        DRC_REQUIRE(candidates[i] >= 1 && candidates[i] <= c->D, "heteroconv_profile_k: candidate %d is %d, D = %d", i,
                    candidates[i], c->D);
        if (candidates[i] > kmax) kmax = candidates[i];
    }
    const int D = c->D;
    const size_t rows = (size_t)(c->Nc > c->Nn ? c->Nc : c->Nn);
    float *vals = nullptr, *H = nullptr, *G = nullptr;
    uint16_t* idx = nullptr;
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    hipStream_t s = nullptr;
    auto body = [&]() -> int {
        DRC_HIP(hipDeviceSynchronize());
        DRC_HIP(hipMalloc((void**)&vals, 4 * rows * kmax + 256));
        DRC_HIP(hipMalloc((void**)&idx, 2 * rows * kmax + 256));
        DRC_HIP(hipMalloc((void**)&G, 4 * rows * kmax + 256));
        DRC_HIP(hipMalloc((void**)&H, 4 * rows * D + 256));
        for (hipEvent_t& e : ev) DRC_HIP(hipEventCreate(&e));
        for (int r = 0; r < 3; ++r) {
            // sources of near and pins are cells, of pinned nets; the upstream gradient of the backward is any
            // dense [M, D] array (the kernels' time does not depend on values): the destination type's embeddings
            const float* Xsrc = (r == 2) ? X_net : X_cell;
            const float* dH = (r == 1) ? X_net : X_cell;
            const int64_t n_src = c->A[r].n_cols;
            int best = -1;
            float best_ms = 0.f;
            for (int i = 0; i < n_candidates; ++i) {
                const int k = candidates[i];
                DRC_TRY(launch_topk(Xsrc, n_src, D, k, vals, idx, s));
                for (int w = 0; w < warmup; ++w) {
                    DRC_TRY(launch_spmm_fwd(&c->A[r], vals, idx, D, k, H, s));
                    DRC_TRY(launch_spmm_bwd(&c->At[r], dH, idx, D, k, G, 0, s));
                }
                DRC_HIP(hipEventRecord(ev[0], s));
                for (int q = 0; q < reps; ++q) DRC_TRY(launch_spmm_fwd(&c->A[r], vals, idx, D, k, H, s));
                DRC_HIP(hipEventRecord(ev[1], s));
                for (int q = 0; q < reps; ++q) DRC_TRY(launch_spmm_bwd(&c->At[r], dH, idx, D, k, G, 0, s));
                DRC_HIP(hipEventRecord(ev[2], s));
                DRC_HIP(hipEventSynchronize(ev[2]));
                float f = 0.f, b = 0.f;
                DRC_HIP(hipEventElapsedTime(&f, ev[0], ev[1]));
                DRC_HIP(hipEventElapsedTime(&b, ev[1], ev[2]));
                ms_fwd[r * n_candidates + i] = f / reps;
                ms_bwd[r * n_candidates + i] = b / reps;
                const float tot = (f + b) / reps;
                if (best < 0 || tot < best_ms || (tot == best_ms && k < candidates[best])) { best = i; best_ms = tot; }
            }
            best_k[r] = candidates[best];
        }
        return DR_OK;
    };
    const int rc = body();
    (void)hipDeviceSynchronize();
    for (hipEvent_t e : ev)
        if (e) (void)hipEventDestroy(e);
    (void)hipFree(vals); (void)hipFree(idx); (void)hipFree(G); (void)hipFree(H);
    return rc;
}

int heteroconv_num_kernels(void) { return kNumKernels; }

const char* heteroconv_kernel_name(int id) { return (id >= 0 && id < kNumKernels) ? kKernelNames[id] : ""; }

int heteroconv_kernel_times(dr_heteroconv* ctx, double* ms_sum, int64_t* launches, int n) {
    DRC_REQUIRE(ctx && ms_sum && launches, "heteroconv_kernel_times: null argument");
    DRC_REQUIRE(n >= kNumKernels, "heteroconv_kernel_times: arrays need heteroconv_num_kernels() entries");
    for (int i = 0; i < n; ++i) { ms_sum[i] = 0.0; launches[i] = 0; }
    DRC_HIP(hipDeviceSynchronize());
    for (TimedLaunch& t : *ctx->timed) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, t.start, t.stop) == hipSuccess) { ms_sum[t.id] += ms; launches[t.id] += 1; }
        if (!t.start_shared) ctx->event_pool->push_back(t.start);
        ctx->event_pool->push_back(t.stop);
    }
    ctx->timed->clear();
    return DR_OK;
}

static int check_weights(const dr_heteroconv_weights* W, const char* fn) {
    DRC_REQUIRE(W != nullptr, "%s: null weights", fn);
    DRC_REQUIRE(W->self_near && W->neigh_near && W->self_pins && W->neigh_pins && W->pinned,
                "%s: null weight matrix", fn);
    DRC_REQUIRE(aligned(W->self_near, 16) && aligned(W->neigh_near, 16) && aligned(W->self_pins, 16) &&
                    aligned(W->neigh_pins, 16) && aligned(W->pinned, 16),
                "%s: weight matrices must be 16-byte aligned", fn);
    return DR_OK;
}

static int check_saved(const dr_heteroconv* c, const dr_heteroconv_saved* S, const char* fn) {
    DRC_REQUIRE(S != nullptr, "%s: null saved", fn);
    DRC_REQUIRE(S->vals_cell && S->idx_cell && S->vals_net && S->idx_net && S->H_near && S->H_pins &&
                    S->H_pinned && S->mask,
                "%s: null buffer in saved", fn);
    DRC_REQUIRE(aligned(S->H_near, 16) && aligned(S->H_pins, 16) && aligned(S->H_pinned, 16) &&
                    aligned(S->mask, 4) && aligned(S->vals_cell, 4) && aligned(S->vals_net, 4),
                "%s: misaligned buffer in saved", fn);
    if (c->k_pins != c->k_near)
        DRC_REQUIRE(S->vals_cell_pins && S->idx_cell_pins && aligned(S->vals_cell_pins, 4),
                    "%s: k_pins != k_near needs saved.vals_cell_pins / idx_cell_pins", fn);
    if (c->k_self != c->k_pinned)
        DRC_REQUIRE(S->vals_net_self && S->idx_net_self && aligned(S->vals_net_self, 4),
                    "%s: k_pins != k_pinned needs saved.vals_net_self / idx_net_self", fn);
    return DR_OK;
}

// The CBSR each use of an embedding reads: a width shared by both uses of a node type shares the buffers.
struct CbsrSets {
    const float *v_near, *v_pins, *v_self, *v_pinned;
    const uint16_t *i_near, *i_pins, *i_self, *i_pinned;
    bool cell_split, net_split;
};
static CbsrSets cbsr_sets(const dr_heteroconv* c, const dr_heteroconv_saved* S) {
    CbsrSets q;
    q.cell_split = c->k_pins != c->k_near;
    q.net_split = c->k_self != c->k_pinned;
    q.v_near = S->vals_cell; q.i_near = S->idx_cell;
    q.v_pinned = S->vals_net; q.i_pinned = S->idx_net;
    q.v_pins = q.cell_split ? S->vals_cell_pins : S->vals_cell;
    q.i_pins = q.cell_split ? S->idx_cell_pins : S->idx_cell;
    q.v_self = q.net_split ? S->vals_net_self : S->vals_net;
    q.i_self = q.net_split ? S->idx_net_self : S->idx_net;
    return q;
}

int heteroconv_fwd(dr_heteroconv* c, const float* X_cell, const float* X_net, const dr_heteroconv_weights* W,
                   float* Y_cell, float* Y_net, const dr_heteroconv_saved* S, void* stream) {
    const LayerFwd g{c, X_cell, X_net, Y_cell, Y_net, S};
    return heteroconv_forward(&g, 1, W, as_stream(stream), ForwardOptions{});
}

int heteroconv_bwd(dr_heteroconv* c, const float* dY_cell, const float* dY_net, const dr_heteroconv_weights* W,
                   const dr_heteroconv_saved* S, float* dX_cell, float* dX_net, const dr_heteroconv_wgrads* dW,
                   void* stream) {
    DRC_REQUIRE(dW && dW->self_near && dW->neigh_near && dW->self_pins && dW->neigh_pins && dW->pinned,
                "heteroconv_bwd: null weight gradient");
    const LayerBwd g{c, dY_cell, dY_net, S, dX_cell, dX_net, *dW};
    return heteroconv_backward(&g, 1, W, as_stream(stream), BackwardOptions{});
}

}  // extern "C"

// Whether each relation gets launches of its own.  Shared launches fill the compute units that the last workgroups of a relation leave
// idle, and random and grid-local gathers pass side by side.  Whole layers, apart / shared, ms: D = 128, 500 000 cells 2.43 / 2.30,
// 700 000 3.45 / 3.32, 1.2 M 6.03 / 5.96 (k = 8 5.41 / 5.36), 2 M 9.70 / 9.67; 1.2 M cells of D = 64 2.93 / 2.85, of D = 96
// 4.99 / 4.86.  The line is where nothing is left of that.  Per-kernel timing needs separate launches.
constexpr int64_t kApartFrom = int64_t(1) << 28;           // elements of a node type's rows
bool drc::heteroconv_relations_apart(const dr_heteroconv* c) {
    if (c->profile || c->overlap == DR_OVERLAP_OFF) return true;
    if (c->overlap == DR_OVERLAP_ON) return false;
    const int64_t rows = c->Nc > c->Nn ? c->Nc : c->Nn;
    return rows * c->D >= kApartFrom;
}

int drc::heteroconv_forward(const LayerFwd* g, int n, const dr_heteroconv_weights* W, hipStream_t s, ForwardOptions opt) {
    // opt.skip_net_output: Y_net is not wanted (last layer of a model whose read-out uses the cells only): the pins
    // module -- its DR-SpMM and its projection -- is not launched, and H_pins / Y_net are left untouched.
    const bool pins_module = !opt.skip_net_output;
    DRC_REQUIRE(n >= 1 && n <= kMaxGraphs, "heteroconv_fwd: %d graphs in one pass", n);
    DRC_TRY(check_weights(W, "heteroconv_fwd"));
    TopkJob tk[2 * kMaxGraphs];
    SpmmFwdJob sp[3 * kMaxGraphs];
    ProjFwdJob pj[kMaxGraphs];
    int n_sp = 0;
    bool apart = false;
    const int D = g[0].c ? g[0].c->D : 0;
    for (int i = 0; i < n; ++i) {
        const LayerFwd& L = g[i];
        dr_heteroconv* c = L.c;
        DRC_REQUIRE(c != nullptr, "heteroconv_fwd: null context");
        DRC_REQUIRE(L.X_cell && L.X_net && L.Y_cell && L.Y_net, "heteroconv_fwd: null tensor");
        DRC_REQUIRE(aligned(L.X_cell, 16) && aligned(L.X_net, 16) && aligned(L.Y_cell, 16) && aligned(L.Y_net, 16),
                    "heteroconv_fwd: tensors must be 16-byte aligned");
        const dr_heteroconv_saved* S = L.S;
        DRC_TRY(check_saved(c, S, "heteroconv_fwd"));
        c->chain_stop = nullptr;
        apart = apart || heteroconv_relations_apart(c);
        const CbsrSets q = cbsr_sets(c, S);
        // A node type that is read at two widths is selected at both in one pass over its embeddings.
        tk[2 * i] = TopkJob{L.X_net, c->Nn, c->k_pinned, S->vals_net, S->idx_net, c->k_self,
                            q.net_split ? S->vals_net_self : nullptr, q.net_split ? S->idx_net_self : nullptr};
        tk[2 * i + 1] = TopkJob{L.X_cell, c->Nc, c->k_near, S->vals_cell, S->idx_cell, c->k_pins,
                                q.cell_split ? S->vals_cell_pins : nullptr, q.cell_split ? S->idx_cell_pins : nullptr};
        if (pins_module) sp[n_sp++] = SpmmFwdJob{&c->A[1], q.v_pins, q.i_pins, c->k_pins, S->H_pins};     // the high-fanout nets start first
        sp[n_sp++] = SpmmFwdJob{&c->A[2], q.v_pinned, q.i_pinned, c->k_pinned, S->H_pinned};
        sp[n_sp++] = SpmmFwdJob{&c->A[0], q.v_near, q.i_near, c->k_near, S->H_near};
        pj[i] = ProjFwdJob{c->Nc, pins_module ? c->Nn : 0, q.v_near, q.i_near, c->k_near, S->H_near, S->H_pinned, L.Y_cell, S->mask,
                           q.v_self, q.i_self, c->k_self, S->H_pins, L.Y_net};
    }
    if (!(apart && n == 1)) {
        DRC_TRY(launch_topks(tk, 2 * n, D, s));
        DRC_TRY(launch_spmm_fwds(sp, n_sp, D, s));
        return launch_proj_fwd(pj, n, *W, D, opt.relu_out, s);
    }
    // One launch per relation: every D-ReLU output is gathered right after it is written, the random relations (pinned,
    // pins) before the grid-local one, the streaming projections last.
    dr_heteroconv* c = g[0].c;
    { ScopedTiming tm(c, kTopkNet, s); DRC_TRY(launch_topks(&tk[0], 1, D, s)); }
    { ScopedTiming tm(c, kFwdPinned, s); DRC_TRY(launch_spmm_fwds(&sp[n_sp - 2], 1, D, s)); }
    { ScopedTiming tm(c, kTopkCell, s); DRC_TRY(launch_topks(&tk[1], 1, D, s)); }
    if (pins_module) { ScopedTiming tm(c, kFwdPins, s); DRC_TRY(launch_spmm_fwds(&sp[0], 1, D, s)); }
    { ScopedTiming tm(c, kFwdNear, s); DRC_TRY(launch_spmm_fwds(&sp[n_sp - 1], 1, D, s)); }
    ProjFwdJob part = pj[0];
    part.Nn = 0;
    { ScopedTiming tm(c, kProjCell, s); DRC_TRY(launch_proj_fwd(&part, 1, *W, D, opt.relu_out, s)); }
    part = pj[0];
    part.Nc = 0;
    if (pins_module) { ScopedTiming tm(c, kProjPins, s); DRC_TRY(launch_proj_fwd(&part, 1, *W, D, opt.relu_out, s)); }
    return DR_OK;
}

static int backward_pass(const LayerBwd* g, int n, const dr_heteroconv_weights* W, hipStream_t s, BackwardOptions opt) {
    // opt.skip_dx: only the weight gradients are wanted (first layer of a model: nobody reads the gradient of the
    // input features), so the projections to dH, the transposed SpMMs and the dX write-outs are not launched.
    // opt.dy_net_zero: dY_net holds zeros (last layer of a model whose loss reads the cells only): everything it
    // would feed is zero, so the pins module's dH, transposed SpMM and weight gradients are not computed.
    const bool need_dx = !opt.skip_dx, net_zero = opt.dy_net_zero;
    DRC_REQUIRE(n >= 1 && n <= kMaxGraphs, "heteroconv_bwd: %d graphs in one pass", n);
    DRC_TRY(check_weights(W, "heteroconv_bwd"));
    WgradJob wj[2 * kMaxGraphs];
    ProjBwdJob pj[kMaxGraphs];
    SpmmBwdJob first[3 * kMaxGraphs], then[kMaxGraphs];      // compact sums; `then` adds to what `first` wrote
    SpmmDenseJob dj[2 * kMaxGraphs];
    int n_first = 0, n_then = 0;
    bool apart = false;
    const int D = g[0].c ? g[0].c->D : 0;
    for (int i = 0; i < n; ++i) {
        const LayerBwd& L = g[i];
        dr_heteroconv* c = L.c;
        DRC_REQUIRE(c != nullptr, "heteroconv_bwd: null context");
        DRC_REQUIRE(L.dY_cell && L.dY_net && (!need_dx || (L.dX_cell && L.dX_net)), "heteroconv_bwd: null tensor");
        DRC_REQUIRE(aligned(L.dY_cell, 16) && aligned(L.dY_net, 16) && aligned(L.dX_cell, 16) && aligned(L.dX_net, 16),
                    "heteroconv_bwd: misaligned tensor");
        const dr_heteroconv_saved* S = L.S;
        DRC_TRY(check_saved(c, S, "heteroconv_bwd"));
        c->chain_stop = nullptr;
        apart = apart || heteroconv_relations_apart(c);
        const CbsrSets q = cbsr_sets(c, S);
        wj[2 * i] = WgradJob{c->Nc, L.dY_cell, S->mask, S->H_near, S->H_pinned, q.v_near, q.i_near, c->k_near,
                             L.dW.neigh_near, L.dW.self_near, L.dW.pinned, c->wg_scratch[0]};
        wj[2 * i + 1] = WgradJob{net_zero ? 0 : c->Nn, L.dY_net, nullptr, S->H_pins, nullptr, q.v_self, q.i_self, c->k_self,
                                 L.dW.neigh_pins, L.dW.self_pins, nullptr, c->wg_scratch[1]};
        if (!need_dx) continue;
        float* const dH_pins = c->dH + (size_t)c->Nc * D;
        pj[i] = ProjBwdJob{c->Nc, net_zero ? 0 : c->Nn, L.dY_cell, S->mask, c->dH, c->dH_pinned, q.i_near, c->k_near, c->S_cell,
                           L.dY_net, dH_pins, q.i_self, c->k_self, c->S_net};
        // ---- cells: self term and near at the near selection, pins at its own (the same where the widths coincide) ----
        const float* g_near = opt.gate_inputs ? q.v_near : nullptr;
        const float* g_pins = opt.gate_inputs ? q.v_pins : nullptr;
        const bool split = q.cell_split && !net_zero;
        const dr_csr* pins_t = net_zero ? nullptr : &c->At[1];
        SpmmDenseJob& jc = dj[2 * i];
        jc = SpmmDenseJob{};
        jc.n_rows = c->Nc; jc.dX = L.dX_cell; jc.dH = c->dH;
        const CompactPiece near_piece{q.i_near, c->k_near, c->S_cell, g_near};
        const bool staged = c->near_plan != nullptr;
        const bool near_apart = staged || split || c->k_near > kDenseMaxK;   // near's sum joins the self term in S_cell first
        if (near_apart && !staged) first[n_first++] = SpmmBwdJob{&c->At[0], c->dH, q.i_near, c->k_near, c->S_cell, 1};
        if (!split) {
            if (c->k_near <= kDenseMaxK) {
                jc.idx = q.i_near; jc.k = c->k_near; jc.init = c->S_cell; jc.gate = g_near;
                if (near_apart) { jc.At2 = pins_t; jc.dH = dH_pins; }
                else { jc.At = &c->At[0]; jc.At2 = pins_t; jc.col2_off = (int)c->Nc; }
            } else {
                if (pins_t) then[n_then++] = SpmmBwdJob{pins_t, dH_pins, q.i_near, c->k_near, c->S_cell, 1};
                jc.more[0] = near_piece;
            }
        } else {
            jc.more[0] = near_piece;
            if (c->k_pins <= kDenseMaxK) {
                jc.idx = q.i_pins; jc.k = c->k_pins; jc.gate = g_pins;
                jc.At2 = pins_t; jc.dH = dH_pins;
            } else {
                first[n_first++] = SpmmBwdJob{pins_t, dH_pins, q.i_pins, c->k_pins, c->G_pins, 0};
                jc.more[1] = CompactPiece{q.i_pins, c->k_pins, c->G_pins, g_pins};
            }
        }
        // ---- nets: pinned at its selection, the pins self term at its own ----
        const float* g_self = opt.gate_inputs ? q.v_self : nullptr;
        const float* g_pinned = opt.gate_inputs ? q.v_pinned : nullptr;
        SpmmDenseJob& jn = dj[2 * i + 1];
        jn = SpmmDenseJob{};
        jn.n_rows = c->Nn; jn.dX = L.dX_net; jn.dH = c->dH_pinned;
        if (c->k_pinned <= kDenseMaxK) {
            jn.At = &c->At[2]; jn.idx = q.i_pinned; jn.k = c->k_pinned; jn.gate = g_pinned;
            if (!net_zero && !q.net_split) jn.init = c->S_net;
        } else {
            float* const to = q.net_split ? c->G_pinned : c->S_net;
            first[n_first++] = SpmmBwdJob{&c->At[2], c->dH_pinned, q.i_pinned, c->k_pinned, to, (!q.net_split && !net_zero) ? 1 : 0};
            jn.more[1] = CompactPiece{q.i_pinned, c->k_pinned, to, g_pinned};
        }
        if (q.net_split && !net_zero) jn.more[0] = CompactPiece{q.i_self, c->k_self, c->S_net, g_self};
    }
    const bool alone = apart && n == 1;
    // The weight gradients come first: what the projections write is then gathered right away.
    if (!alone) {
        if (!need_dx) return launch_wgrads(wj, 2 * n, D, s);
        PendingSums sums{};
        DRC_TRY(launch_dense_bwd(wj, pj, n, *W, D, g[0].c->wg_sums, &sums, s));
        for (int i = 0; i < n; ++i)
            if (g[i].c->near_plan)
                DRC_TRY(launch_spmm_bwd_planned(g[i].c->near_plan, g[i].c->dH, cbsr_sets(g[i].c, g[i].S).i_near, g[i].c->k_near, g[i].c->S_cell, 1, s));
        if (n_first) DRC_TRY(launch_spmm_bwds(first, n_first, D, s));
        if (n_then) DRC_TRY(launch_spmm_bwds(then, n_then, D, s));
        DRC_TRY(launch_spmm_dense(dj, 2 * n, D, s, &sums));
        return launch_pending_sums(sums, s);
    }
    dr_heteroconv* c = g[0].c;
    { ScopedTiming tm(c, kWgCell, s); DRC_TRY(launch_wgrads(&wj[0], 1, D, s)); }
    { ScopedTiming tm(c, kWgPins, s); DRC_TRY(launch_wgrads(&wj[1], 1, D, s)); }
    if (!need_dx) return DR_OK;
    ProjBwdJob part = pj[0];
    part.Nc = 0;
    if (part.Nn) { ScopedTiming tm(c, kDhPins, s); DRC_TRY(launch_proj_bwd(&part, 1, *W, D, s)); }
    part = pj[0];
    part.Nn = 0;
    { ScopedTiming tm(c, kDhCell, s); DRC_TRY(launch_proj_bwd(&part, 1, *W, D, s)); }
    { ScopedTiming tm(c, kBwdPinned, s); DRC_TRY(launch_spmm_dense(&dj[1], dj[1].At ? 1 : 0, D, s)); }
    if (c->near_plan) {
        ScopedTiming tm(c, kBwdNear, s);
        DRC_TRY(launch_spmm_bwd_planned(c->near_plan, c->dH, cbsr_sets(c, g[0].S).i_near, c->k_near, c->S_cell, 1, s));
    }
    if (n_first) { ScopedTiming tm(c, kBwdNear, s); DRC_TRY(launch_spmm_bwds(first, n_first, D, s)); }
    if (n_then) { ScopedTiming tm(c, kBwdPins, s); DRC_TRY(launch_spmm_bwds(then, n_then, D, s)); }
    { ScopedTiming tm(c, dj[0].At ? kBwdNearPins : kBwdPins, s); DRC_TRY(launch_spmm_dense(&dj[0], dj[1].At ? 1 : 2, D, s)); }
    return DR_OK;
}

void drc::heteroconv_ordered_on(dr_heteroconv* c, hipStream_t s) {
    c->last_stream = s;
    c->has_last = true;
}

void drc::heteroconv_hand_over(dr_heteroconv* c, hipStream_t from, hipStream_t to) {
    if (!c->has_last || c->last_stream == from) heteroconv_ordered_on(c, to);
}

int drc::heteroconv_backward(const LayerBwd* g, int n, const dr_heteroconv_weights* W, hipStream_t s, BackwardOptions opt) {
    bool plain = true;
    for (int i = 0; i < n; ++i) plain = plain && (!g[i].c || (g[i].c->has_last && g[i].c->last_stream == s && !g[i].c->many_streams));
    if (plain) return backward_pass(g, n, W, s, opt);
    // A captured pass is ordered by the graph it becomes part of: events of the world outside do not belong in it.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    DRC_HIP(hipStreamIsCapturing(s, &capture));
    if (capture != hipStreamCaptureStatusNone) return backward_pass(g, n, W, s, opt);
    for (int i = 0; i < n; ++i) {
        dr_heteroconv* const c = g[i].c;
        if (!c) continue;
        if (c->has_last && c->last_stream != s) {
            if (c->end_recorded) DRC_HIP(hipStreamWaitEvent(s, c->end, 0));
            else DRC_HIP(hipDeviceSynchronize());
            c->many_streams = true;
        }
        heteroconv_ordered_on(c, s);
        c->end_recorded = false;
    }
    DRC_TRY(backward_pass(g, n, W, s, opt));
    for (int i = 0; i < n; ++i)
        if (g[i].c->many_streams) {
            DRC_HIP(hipEventRecord(g[i].c->end, s));
            g[i].c->end_recorded = true;
        }
    return DR_OK;
}
