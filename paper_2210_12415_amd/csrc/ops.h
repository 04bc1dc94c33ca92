// Shared between ops.hip (conv/gemm entry points) and tune.cpp.
#pragma once

#include <functional>

#include "dconv.h"

namespace alt {

// What the kernels over filter taps add to a 2-D problem: a depth direction, whose taps lie beside the channels in a filter
// row ((r, s), (t, c): the filter alt_conv3d packs), and the output phases of a transposed convolution in its sub-pixel form.
// All zero for an ordinary problem.
struct Volume {
    int32_t T, D, OD, stride_d, pad_d, dil_d;   // T = 0: an ordinary problem
    int32_t sd, sh, sw;                         // phases per direction (1: none); then per direction:
    int32_t pad[3], taps[3];                    // the operator's own padding and the taps of one phase
};

// One conv/gemm call reduced to what the implicit-GEMM kernels need.
struct Problem {
    IgemmParams p;
    int dtype;
    bool a_vec, a_trans, b_vec, b_trans;   // loaders the operand layouts admit (gather always works)
    bool spatial_split, spatial_ok;
    int64_t x_elems, w_elems;              // elements of one batch entry of each operand
    int64_t groups;                        // convolution groups (1 for ordinary problems and products)
    bool depthwise;                        // groups = C = K: runs on dwconv.hip, p describes the whole tensors
    Volume v;
};

// A 3-D or transposed convolution as the kernels over filter taps read it: `f` the merged or depth-unfolded 2-D problem, over
// whose weights they run, xs and ys the extents of the tensors where they lie.
struct TapsCall {
    alt_conv_desc_t f;
    int64_t xs[4], ys[4];
    int64_t C, K;                          // channels of a tap, output channels of a phase
    Volume v;
};

extern const int kSplitFactors[];
int igemm_num_splits();
int igemm_variant_count();
std::string igemm_variant_name(int variant);
void igemm_analyse(Problem *pb);
bool igemm_applicable(const Problem &pb, const IgemmLaunch &k, int splitk, std::string *why);
size_t igemm_workspace(const Problem &pb, int splitk);
double igemm_estimate(const Problem &pb, const IgemmLaunch &k, const IgemmParams &p, size_t lds);
// Every variant that runs the problem within the workspace, with its estimate (counters = false: those that need no arrival counters)
void igemm_for_each(const Problem &pb, size_t ws_limit, bool counters, const std::function<void(int variant, double estimate)> &seen);
int igemm_default_variant(const Problem &pb, size_t ws_limit, bool counters = true);
// A tile kernel's launch worked out for one problem; the operands' addresses are filled in by every call.
struct TileLaunch {
    int variant = -1;                      // -1: nothing yet
    size_t lds = 0;
    DconvParams d;
};
// (*no_counters: the variant's slices need arrival counters and no set of them is free for the stream; kept: where the same
// problem's launch is kept between calls)
alt_status_t igemm_run(alt_handle_t h, const Problem &pb, int variant, void *workspace, size_t ws_bytes,
                       hipStream_t st, bool *no_counters = nullptr, TileLaunch *kept = nullptr);

// dconv.hip
bool dconv_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes,
                 std::string *why);
void dconv_splitk_state(int *slots_bound, int *counters_nonzero);
hipError_t dconv_run(const IgemmLaunch &k, DconvParams d, size_t lds, float *partial, hipStream_t st);

// ops.hip: device address of alt_conv2d_static's workspace array on the current device
hipError_t static_scratch(void **out);

// dwconv.hip
alt_status_t depthwise_run(alt_handle_t h, const Problem &pb, int64_t N, int64_t C, hipStream_t st);

// eltwise.hip
alt_status_t eltwise_add(alt_handle_t h, int dtype, int64_t numel, const void *a, const void *b, void *y, int relu,
                         hipStream_t st);

// ops.hip: runs the call on a kernel over filter taps and says so in *done, or leaves it alone (a layout, size or alignment these
// kernels do not take, or a variant of the 2-D problem asked for, by number or by a tuned entry).  ws_2d: bytes of the workspace
// the 2-D problem would have for itself, negative if its operands do not fit.
alt_status_t taps_run(alt_handle_t h, const TapsCall &c, const void *x, const void *w, const float *bias, void *y, void *workspace,
                      size_t ws_bytes, int64_t ws_2d, hipStream_t st, bool *done);
// Bytes of workspace that the kernel taps_run would choose wants for itself (0 where it would leave the call alone).
size_t taps_workspace(alt_handle_t h, const TapsCall &c);

alt_status_t conv_problem(alt_handle_t h, const alt_conv_desc_t *d, const void *x, const void *w,
                          const float *bias, void *y, Problem *pb);
alt_status_t gemm_problem(alt_handle_t h, const alt_gemm_desc_t *d, const void *A, const void *B, void *C,
                          Problem *pb);

// t2d.hip: the kernels that put the output phases of a sub-pixel transposed convolution into place
alt_status_t phase_shuffle(alt_handle_t h, const alt_layout_t *layout, int64_t N, int64_t K, int64_t ODq, int64_t OHq, int64_t OWq,
                           int sd, int sh, int sw, int elsz, const void *src, void *dst, hipStream_t st);
alt_status_t phase_bias(alt_handle_t h, const float *bias, float *out, int64_t K, int64_t n, hipStream_t st);

alt_status_t transform_bound(alt_handle_t h, int elsz, const BoundLayout &ls, const void *src,
                             const BoundLayout &ld, void *dst, hipStream_t st);

}  // namespace alt
