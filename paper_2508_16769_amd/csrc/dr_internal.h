// Internal declarations shared by the HIP translation units of libdrcgnn (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstddef>
#include <cstdint>
#include <cstdio>

#include "dr_circuitgnn.h"
#include "launch_shape.h"
#include "per_device.h"

namespace drc {

constexpr int kWave = 64;      // CDNA wavefront width
constexpr int kNumXcd = 8;     // MI355X: 8 accelerator complex dies, one L2 each

// thread-local error text ------------------------------------------------------------------------
void set_error(const char* fmt, ...);
int fail(int code, const char* fmt, ...);
int hip_fail(hipError_t e, const char* what);

#define DRC_HIP(call)                                                   \
    do {                                                                \
        hipError_t drc_e__ = (call);                                    \
        if (drc_e__ != hipSuccess) return ::drc::hip_fail(drc_e__, #call); \
    } while (0)

#define DRC_REQUIRE(cond, ...)                                          \
    do {                                                                \
        if (!(cond)) return ::drc::fail(DR_ERR_INVALID_ARG, __VA_ARGS__); \
    } while (0)

#define DRC_TRY(expr)                  \
    do {                               \
        int drc_rc__ = (expr);         \
        if (drc_rc__) return drc_rc__; \
    } while (0)

int check_csr(const dr_csr* A, const char* name, bool need_vals);
inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }

// Workgroups are dealt to the XCDs round-robin by workgroup id.  Remap so that each XCD walks one
// contiguous range of logical tiles (neighbouring tiles share gathered rows in that XCD's L2).
// `per_xcd` = ceil(n_tiles / kNumXcd); launch per_xcd * kNumXcd workgroups and drop ids >= n_tiles.
__device__ __forceinline__ int xcd_contiguous_tile(int wg, int per_xcd) {
    return (wg % kNumXcd) * per_xcd + wg / kNumXcd;
}

// launchers (host side, argument checks already done by the ABI layer) ------------------------------
int launch_topk(const float* X, int64_t n, int D, int k, float* vals, uint16_t* idx, hipStream_t s);
// Several embedding matrices in one launch; vals2 != nullptr: the same rows are selected at a second width in the same pass.
struct TopkJob {
    const float* X;
    int64_t n;
    int k;
    float* vals;
    uint16_t* idx;
    int k2;
    float* vals2;
    uint16_t* idx2;
};
int launch_topks(const TopkJob* jobs, int n, int D, hipStream_t s);
// The dense products halve their operands: kUnscale takes a sum of products back.
constexpr float kUnscale = 4.0f;
// A weight gradient whose partial sums wait in scratch memory: dst[at] = kUnscale * sum over i < n of src[i * count + at], at < count.
struct PartialSum {
    const float* src;
    float* dst;
    int n, count;
};
// Weight gradients that a later launch on the same stream is to sum up; the table is written by the launch that writes the partials.
struct PendingSums {
    const PartialSum* table;      // device memory
    int n, count;                 // n = 0: nothing is pending
};
// DR-SpMM.  A job is one relation; jobs of one call may share launches and run side by side.
constexpr int kMaxSegs = 18;     // relations per launch (their descriptors travel as kernel arguments)
struct SpmmFwdJob {
    const dr_csr* A;
    const float* xs_vals;
    const uint16_t* xs_idx;
    int k;
    float* H;
};
struct SpmmBwdJob {
    const dr_csr* At;
    const float* dH;
    const uint16_t* xs_idx;
    int k;
    float* dXs;
    int accumulate;
};
struct CompactPiece {            // gradient on a selection [rows, k]; entries whose gate value is not positive are dropped
    const uint16_t* idx;
    int k;
    const float *vals, *gate;     // gate may be null
};
// Input gradient of one kind of source rows, written dense: dX[row, :] = 0 except at the columns of the row's selection
// idx[row, :], where it is  init[row, t] + sum over the row's edges of At (gathering dH rows) and of At2 (gathering dH rows
// col2_off further on); entries whose gate value is not positive are zero.  Up to two further compact pieces are added at
// their own columns.  At, At2, init, gate and the pieces may be absent (k = 0: no selection of its own).
struct SpmmDenseJob {
    int64_t n_rows;
    const dr_csr *At, *At2;
    int col2_off;
    const float* dH;              // at least one row is readable
    const uint16_t* idx;
    int k;
    float* dX;
    const float *init, *gate;
    CompactPiece more[2];
};
constexpr int kDenseMaxK = 64;   // one window of compact slots
// `pending` (may be null): summed up by the last launch of these; what no launch took stays pending.
int launch_spmm_dense(const SpmmDenseJob* jobs, int n, int D, hipStream_t s, PendingSums* pending = nullptr);    // n <= 64
int launch_spmm_fwds(const SpmmFwdJob* jobs, int n, int D, hipStream_t s);       // n <= 64
int launch_spmm_bwds(const SpmmBwdJob* jobs, int n, int D, hipStream_t s);       // n <= 64
int launch_spmm_fwd(const dr_csr* A, const float* xs_vals, const uint16_t* xs_idx, int D, int k, float* H,
                    hipStream_t s);
int launch_spmm_bwd(const dr_csr* At, const float* dH, const uint16_t* xs_idx, int D, int k, float* dXs,
                    int accumulate, hipStream_t s);
int launch_topk_ranked(const float* X, int64_t n, int D, int k, float* vals, uint16_t* idx, hipStream_t s);
int launch_spmm_fwd_adaptive(const dr_csr* A, const float* xr_vals, const uint16_t* xr_idx, int D, const dr_degree_classes* c,
                             float* H, hipStream_t s);
int launch_spmm_bwd_adaptive(const dr_csr* At, const uint8_t* edge_class, const float* dH, const uint16_t* xr_idx, int D,
                             const dr_degree_classes* c, float* dXr, int accumulate, hipStream_t s);
int launch_edge_classes(const dr_csr* At, const int32_t* a_rowptr, const dr_degree_classes* c, uint8_t* out, hipStream_t s);
struct TransposeJob {             // one relation of a set that is transposed by the same launches (each with its own workspace)
    const dr_csr* A;
    int32_t *t_rowptr, *t_colidx;
    float* t_vals;                // may be null (pattern only)
    void* ws;                     // csr_transpose_workspace() bytes, 256-byte aligned
};
size_t csr_transpose_workspace(int64_t n_cols, int64_t nnz);
int launch_csr_transposes(const TransposeJob* jobs, int n, hipStream_t s);
size_t csr_normalize_workspace(int mode, int64_t n_cols, int64_t nnz);
int launch_csr_normalize(int mode, int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t* rowptr,
                         const int32_t* colidx, float* vals_out, void* ws, hipStream_t s);
int launch_csr_normalize_noalloc(int mode, int64_t n_rows, int64_t n_cols, int64_t nnz, const int32_t* rowptr,
                                 const int32_t* colidx, float* vals_out, hipStream_t s);
int launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s);
// DR-SpMM backward with the gathered rows staged in LDS, tile by tile (staged.hip)
int spmm_plan_create(dr_spmm_plan** out, const dr_csr* A, const int32_t* row_order, int D, hipStream_t s);
void spmm_plan_destroy(dr_spmm_plan* p);
int launch_spmm_bwd_planned(const dr_spmm_plan* p, const float* dH, const uint16_t* xs_idx, int k, float* dXs, int accumulate,
                            hipStream_t s);

constexpr int kMaxGraphs = 16;    // graphs per launch (their descriptors travel as kernel arguments)
// elements of a node type's rows from which on it fills the chip: sub-graphs of a batch share no launches, and cells and nets no workgroups
// for their weight gradients
constexpr int64_t kFullLaunch = int64_t(1) << 26;

// shape of a layer context (heteroconv.hip owns the struct)
struct HeteroDims {
    int64_t Nc, Nn;
    int D;
    int k_near, k_pins, k_self, k_pinned;   // D-ReLU widths: cells for near / for pins, nets for the pins self term / for pinned
};
HeteroDims heteroconv_dims(const dr_heteroconv* c);
const dr_csr* heteroconv_relations(const dr_heteroconv* c);
void heteroconv_capacity(const dr_heteroconv* c, int64_t* cells, int64_t* nets);   // what the context's buffers are sized for   // [3] near, pins, pinned as given to the create call
// A context whose buffers are sized for graphs of up to (Nc, Nn, E[near, pins, pinned]); relations are bound later
// (and again) with heteroconv_bind.  keep_workspace: also keep the transpose workspaces, which heteroconv_bind needs.
int heteroconv_create_capacity(dr_heteroconv** ctx, int64_t Nc, int64_t Nn, const int64_t E[3], int32_t D, int32_t k_near,
                               int32_t k_pins, int32_t k_self, int32_t k_pinned, bool keep_workspace);
int heteroconv_bind(dr_heteroconv* c, const dr_csr* near, const dr_csr* pins, const dr_csr* pinned, hipStream_t s);
// heteroconv_fwd / heteroconv_bwd with what a stacked model knows folded in (see ForwardOptions / BackwardOptions).
struct ForwardOptions {
    bool relu_out = false;          // clamp Y_cell and Y_net at zero as they are written (the mask compares raw values)
    bool skip_net_output = false;   // Y_net (and H_pins) are not wanted: the pins module is not evaluated
};
// A layer pass over up to kMaxGraphs graphs that share the weights: a step is one launch for all of them, or a few where their
// relations are more than a launch takes (kMaxSegs: 16 graphs have 48 forward relations, three launches).
struct LayerFwd {
    dr_heteroconv* c;
    const float *X_cell, *X_net;
    float *Y_cell, *Y_net;
    const dr_heteroconv_saved* S;
};
bool heteroconv_relations_apart(const dr_heteroconv* c);     // whether a pass over this graph alone has a launch per relation
int heteroconv_forward(const LayerFwd* g, int n, const dr_heteroconv_weights* W, hipStream_t s, ForwardOptions opt);
struct BackwardOptions {
    bool gate_inputs = false;     // zero dX where the layer's input was not positive (ReLU in front of the layer)
    bool skip_dx = false;         // weight gradients only: dX_cell / dX_net are not written (and may be null)
    bool dy_net_zero = false;     // dY_net is all zeros: what it would feed is not computed (fills instead)
};
struct LayerBwd {
    dr_heteroconv* c;
    const float *dY_cell, *dY_net;
    const dr_heteroconv_saved* S;
    float *dX_cell, *dX_net;
    dr_heteroconv_wgrads dW;
};
int heteroconv_backward(const LayerBwd* g, int n, const dr_heteroconv_weights* W, hipStream_t s, BackwardOptions opt);
// Where a context's last backward pass is: its scratch is used on one stream at a time, and a pass on another one waits.
void heteroconv_ordered_on(dr_heteroconv* c, hipStream_t s);   // whatever it enqueued comes before what follows on s
void heteroconv_hand_over(dr_heteroconv* c, hipStream_t from, hipStream_t to);   // `to` has just been made to wait for `from`
int heteroconv_create_widths(dr_heteroconv** ctx, const dr_csr* near, const dr_csr* pins, const dr_csr* pinned, int32_t D,
                             int32_t k_near, int32_t k_pins, int32_t k_self, int32_t k_pinned);

// dense part of the layer ------------------------------------------------------------------------------
struct ProjFwdJob {               // one graph: Y_cell, mask, and (Nn > 0) Y_net from the saved selections and messages
    int64_t Nc, Nn;               // Nn = 0: the net output is not wanted
    const float* vals_near;
    const uint16_t* idx_near;
    int k_near;
    const float *H_near, *H_pinned;
    float* Y_cell;
    uint8_t* mask;
    const float* vals_self;
    const uint16_t* idx_self;
    int k_self;
    const float* H_pins;
    float* Y_net;
};
int launch_proj_fwd(const ProjFwdJob* jobs, int n, const dr_heteroconv_weights& W, int D, bool relu, hipStream_t s);

struct ProjBwdJob {               // one graph: dH of the three relations and the sampled self-term gradients S [rows, k]
    int64_t Nc, Nn;               // Nn = 0: dY_net is zero
    const float* dY_cell;
    const uint8_t* mask;
    float *dH_near, *dH_pinned;
    const uint16_t* idx_near;
    int k_near;
    float* S_cell;
    const float* dY_net;
    float* dH_pins;
    const uint16_t* idx_self;
    int k_self;
    float* S_net;
};
int launch_proj_bwd(const ProjBwdJob* jobs, int n, const dr_heteroconv_weights& W, int D, hipStream_t s);

struct WgradJob {                 // one node type of one graph; with a mask: cells (three products), without: nets (two)
    int64_t rows;
    const float* dY;
    const uint8_t* mask;
    const float *H1, *H2;
    const float* vals;
    const uint16_t* idx;
    int k;
    float *dW_H1, *dW_cbsr, *dW_H2;
    void* scratch;                // wgrad_scratch_bytes(rows, D, products)
};
size_t wgrad_scratch_bytes(int64_t rows, int D, int products);
int launch_wgrads(const WgradJob* jobs, int n, int D, hipStream_t s);      // n <= 2 * kMaxGraphs
// Weight gradients (cells and nets of each graph in turn) and projections of a backward pass.  The partial sums of the weight gradients
// are left to launch_spmm_dense, or to launch_pending_sums; `table` has room for kSumsPerGraph entries a graph.
constexpr int kSumsPerGraph = 5;
int launch_dense_bwd(const WgradJob* wgrads, const ProjBwdJob* proj, int n, const dr_heteroconv_weights& W, int D, PartialSum* table,
                     PendingSums* pending, hipStream_t s);
int launch_pending_sums(const PendingSums& pending, hipStream_t s);

}  // namespace drc
