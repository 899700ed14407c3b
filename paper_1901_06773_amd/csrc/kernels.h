// Launchers of the gfx950 kernels.  Every launcher checks that its operand shapes
// fit what the kernel and its grid assume and returns hipErrorInvalidValue otherwise;
// nothing here allocates.  Activations NHWC, filters O-H-W-I (K-contiguous rows); `dtype`
// (DT_F32 / DT_BF16 of dtype.h, the values of ACC_F32 / ACC_BF16) is the storage type of
// activations, activation gradients and of the filter copy the kernels read; arithmetic is
// fp32 (bf16 products on the matrix cores accumulate in fp32), weight gradients, batch-norm
// parameters and statistics, biases and the loss are always fp32.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

#include "bn_shape.h"
#include "dgrad_split.h"

namespace acc {

// A weight-gradient reduction that has not been launched yet: dw[i] = part[0][i] + part[1][i]
// + ... (count elements, `splits` parts, in that order).  count == 0: nothing to do.
struct ReduceJob {
  const float* part;
  float* dw;
  size_t count;
  int splits;
};

// A filter to flip and transpose on the side of another launch (storage type of that launch):
// wt[ci][r'][t'][co] = w[co][R-1-r'][S-1-t'][ci].  wt == nullptr: nothing to do.
struct FlipJob {
  const void* w;
  void* wt;
  int cout, cin, r, s;
};

// Optional work of a data-gradient launch for the batch norm (with ReLU) whose output was the
// convolution's input: the result is the gradient of that output, so the launch masks it with
// [y > 0] before storing it and leaves, per block of 32 rows and per channel, the sums of the
// masked gradient g and of g * xhat (xhat = (x - mean) * istd) in sums[2][stride][n_out]
// (floats; stride >= conv_stat_slabs(rows)).  x, y: the batch norm's input and output, laid
// out like the launch's dense output.  sums == nullptr: off.
struct BnBackwardSums {
  const void* x;
  const void* y;
  const float* mean;
  const float* istd;
  float* sums;
  int stride;
};

// A strided data gradient: the residue classes of dgrad_split(), and the filter w[cout][r][s][cin] their sub-filters come from.
struct DgradSplit {
  const void* w;
  int cout, cin, r, s, stride;
  const DgradPart* parts;
  int count;
};

// Implicit-GEMM view of a convolution-like gather:
//   out[m][n] (+)= sum_{r,t,c} in[img, p*stride+r-pad, q*stride+t-pad, c] * w[n][(r,t,c)]
// with row m = (img, p, q) over a P x Q grid (columns use pad + pad_dx).  The result row is
// written to pixel (out_y0 + p*out_stride, out_x0 + q*out_stride) of an out_h x out_w image
// with `n_out` channels.
struct ConvGeom {
  const void* in;           // dtype
  const void* w;            // dtype
  void* out;                // dtype
  int dtype;
  int n_img, h, wd, c;      // input image size and channels
  int p, q;                 // rows enumerate n_img x p x q positions
  int n_out;                // GEMM N (output channels)
  int r, s, stride, pad;
  int pad_dx;               // column padding is pad + pad_dx (>= 0)
  int out_h, out_w, out_stride;
  int out_y0, out_x0;       // first output pixel
  int accumulate;           // out += result
  const float* bias;        // optional: + bias[n] (fp32), then
  int relu;                 // ... max(., 0) if set; both only without accumulate
  // Optional side jobs: extra workgroups appended to the launch add up the parts of a weight
  // gradient, and / or write the flipped, transposed filter that a later data gradient needs
  // (independent data; saves launches of their own).
  ReduceJob side;
  FlipJob flip;
  // Optional (fp32 storage, plain dense output): per-channel sums of the result and of its
  // square over every block of 32 rows, as the batch norm that follows wants them:
  // stats[0][b][n] = sum, stats[1][b][n] = sum of squares, b < conv_stat_slabs(rows), layout
  // float[2][stats_stride][n_out] with stats_stride >= conv_stat_slabs(rows).
  float* stats;
  int stats_stride;
  BnBackwardSums bnb;   // fp32 storage, plain dense output, no accumulation
  // Optional (host memory, read by conv_igemm only): the launch is a strided data gradient as a whole.  conv_igemm writes
  // the sub-filter of every part to w + its wt_offset (w is then a workspace) and runs the parts; p .. pad_dx, the
  // output's stride and first pixel come from them.
  const DgradSplit* split;
  // Optional (1x1 filters, and with bf16 storage all): the same filter as w[c][taps, the last first][n], the layout a data gradient finds it in: w[k][n] of
  // 1x1.  bf16: read where w is null and conv_igemm_bf16_takes() says so; fp32:  conv_igemm_rows_takes() says
  // whether the launch reads it, and w is then not read and may be null.  A caller that asks with w null would need a launch of
  // its own to write it, and the answer counts that.
  const void* w_kn;
};
// Number of 32-row blocks conv_igemm writes sums for (2 per 64-row tile).
inline long conv_stat_slabs(long rows) { return ((rows + 63) / 64) * 2; }
// Partial sums a convolution launch has left for a batch norm: float part[2][stride][c], `slabs` of
// them valid (each the fp32 sum over one block of 32 rows).
struct BnSums {
  const float* part;
  int slabs, stride;
};

// Optional probe of one launch: which template instance ran (index into conv_variant_name(); `kernel` names it with its
// tile) and, when the two events are set, timestamps recorded directly around the main kernel.  dry: every check and choice
// is made, nothing is launched.
struct LaunchProbe {
  int variant = -1;
  hipEvent_t before = nullptr, after = nullptr;
  const char* kernel = nullptr;
  bool dry = false;
};
hipError_t conv_igemm(const ConvGeom& g, hipStream_t st, LaunchProbe* probe = nullptr);
// The kernels for bf16 storage (conv_igemm_bf16.hip): whether they take this launch (a
// function of the shape and the alignment only), and the launch itself; conv_igemm() routes to it.
bool conv_igemm_bf16_takes(const ConvGeom& g, long M, long K);
hipError_t conv_igemm_bf16(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe);
// fp32 products on the bf16 matrix cores (conv_igemm_x3.hip): as above.
bool conv_igemm_x3_takes(const ConvGeom& g, long M, long K);
hipError_t conv_igemm_x3(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe);
// Whether the direct kernel with the fp32 instruction is predicted to be the faster one for a launch that both take.
bool conv_igemm_x3_slower(const ConvGeom& g, long M, long K);
// The faster of the two, predicted (microseconds).
double conv_igemm_x3_us(const ConvGeom& g, long M, long K);
// The direct fp32 kernel runs two groups of waves per tile: at most one tile per compute unit and at least eight chunks of 32
// values of K (a function of the shape only).
inline bool conv_igemm_two_groups(const ConvGeom& g, long M, long K) {
  return !(g.bias || g.relu) && ((M + 63) / 64) * ((g.n_out + 63) / 64) <= 256 && K >= 256;
}
// Few rows and a long reduction (conv_rows.hip): as above; with g.w_kn set, whether the launch reads that.
bool conv_igemm_rows_takes(const ConvGeom& g, long M, long K);
hipError_t conv_igemm_rows(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe);
// The parts of a strided data gradient in one launch, where that is the faster way (a function of the shapes only).
bool conv_igemm_x3_parts_takes(const ConvGeom* parts, int n);
hipError_t conv_igemm_x3_parts(const ConvGeom* parts, int n, hipStream_t st, LaunchProbe* probe);
// A handful of input channels (conv_smallc.hip): as above.
bool conv_smallc_takes(const ConvGeom& g, long M);
hipError_t conv_smallc_fwd(const ConvGeom& g, hipStream_t st, LaunchProbe* probe);
// Callers see these numbers (acc_get_launch_profile): one keeps its kernel, new ones go to the end.  0 was a kernel that is gone, 15 is none.
enum { V_IGEMM_GENERIC = 1, V_WGRAD_FAST, V_WGRAD_GENERIC, V_IGEMM_DIRECT, V_WGRAD_DIRECT, V_WGRAD_BF16, V_IGEMM_BF16, V_IGEMM_DIRECT_2G,
       V_IGEMM_X3, V_IGEMM_X3_WINDOW, V_IGEMM_X3_DEEP, V_WGRAD_X3, V_SMALLC_FWD, V_SMALLC_WGRAD,
       V_IGEMM_ROWS = 16, V_COUNT };
const char* conv_variant_name(int v);

// dw[co][(r,t,ci)] = sum_{img,p,q} dy[img,p,q,co] * x[img, p*stride+r-pad, q*stride+t-pad, ci]
struct WgradGeom {
  const void* x;            // dtype
  const void* dy;           // dtype
  float* dw;                // fp32
  int dtype;
  int n_img, h, wd, cin;
  int p, q, cout;
  int r, s, stride, pad;
  float* workspace;         // split-K partials, workspace_bytes of them: at least wgrad_workspace_least() (may be null if 0)
  size_t workspace_bytes;
  // Optional side job: extra workgroups appended to the launch write the flipped and
  // transposed filter wt[ci][r'][t'][co] = w[co][R-1-r'][S-1-t'][ci] of this layer (the data
  // gradient that follows needs it).  Both null: no side job.
  const void* flip_w;       // dtype
  void* flip_wt;            // dtype
  // Optional side job: extra workgroups add up the parts of an earlier weight gradient.
  ReduceJob side;
};
// Scratch for the parts of a weight gradient.  dtype: DT_F32 / DT_BF16 (the two storage types cut the minibatch range
// differently), or -1 = the larger of the two.  _bytes: as many parts as are fastest for the call alone; _least: the fewest the
// call works with.  An iteration's plan counts with the fewest: its scratch lies in the budget, and beside the data gradients, on a
// stream of its own, more parts gain nothing (ResNet-50, 32 images, 9560 us with, 9532 without).  How a shape is cut,
// and with it the bits of the result, depends on the shape and on which of the two sizes is there.
size_t wgrad_workspace_least(int n_img, int p, int q, int cin, int cout, int r, int s, int dtype);
size_t wgrad_workspace_bytes(int n_img, int p, int q, int cin, int cout, int r, int s, int dtype);
// If `deferred` is given and the gradient is split over the minibatch, the reduction of the
// parts is not launched but described there (the caller appends it to a later launch or
// runs reduce_parts); otherwise dw is complete when the stream reaches the end of this call.
hipError_t conv_wgrad(const WgradGeom& g, hipStream_t st, LaunchProbe* probe = nullptr,
                      ReduceJob* deferred = nullptr);
// The kernel for fp32 storage on the bf16 matrix cores (conv_wgrad_x3.hip): how it cuts a shape (tile of 64*wt
// squared, steps of 16 positions per part), and the launch; conv_wgrad() routes to it.
struct WgradX3Cfg {
  int wt, tiles_co, tiles_j, splits, steps_per_split;
};
WgradX3Cfg wgrad_x3_choose(long Mrows, int cin, int cout, int r, int s, int max_splits);
hipError_t conv_wgrad_x3(const WgradGeom& g, const WgradX3Cfg& c, int Mrows, int J, float* out, size_t count, hipStream_t st);
// The kernel for bf16 storage (conv_wgrad_bf16.hip): how it cuts a shape (pixels: of the input), with max_splits
// parts at most, the name of the tiling, and the launch.
struct WgradBf16Cfg {
  int kind, tiles_co, tiles_j, splits, chunks_per_split;
};
WgradBf16Cfg wgrad_bf16_choose(long Mrows, long pixels, int cin, int cout, int r, int s, int max_splits);
const char* wgrad_bf16_name(const WgradGeom& g, const WgradBf16Cfg& c);
hipError_t conv_wgrad_bf16(const WgradGeom& g, const WgradBf16Cfg& c, int Mrows, int J, float* out, size_t count, hipStream_t st);
// The kernel for a handful of input channels (conv_smallc.hip): parts it cuts the reduction into (0: the shape is not
// its; a function of what wgrad_workspace_bytes() knows), whether it takes a launch, and the launch.
int wgrad_smallc_splits(long Mrows, int cin, int cout, int r, int s, int dtype);
bool conv_wgrad_smallc_takes(const WgradGeom& g);
hipError_t conv_wgrad_smallc(const WgradGeom& g, int splits, float* out, size_t count, hipStream_t st);
hipError_t reduce_parts(const ReduceJob& job, hipStream_t st);

// wt[ci][r'][t'][co] = w[co][R-1-r'][S-1-t'][ci]  (filter of the transposed convolution)
hipError_t filter_flip_transpose(const void* w, void* wt, int cout, int cin, int r, int s, int dtype,
                                 hipStream_t st);

// The sub-filters of all residue classes of a strided data gradient (dgrad_split.h), each written at wt + its wt_offset.
hipError_t filter_gather_transpose(const DgradSplit& d, void* wt, int dtype, hipStream_t st);

// Batch norm over rows x c (NHWC flattened).  workspace: bn_workspace_bytes(c).
// x, res, y, dy, dx, g_out: dtype; gamma, beta, mean, istd, dgamma, dbeta: fp32.
size_t bn_workspace_bytes(int c);
// ready_sums (may be null): the partial sums of x and x*x are already there (conv_igemm wrote
// them, ConvGeom::stats) and are not computed again.
hipError_t bn_forward(const void* x, const float* gamma, const float* beta, const void* res,
                      void* y, float* mean, float* istd, long rows, int c, int relu, float eps,
                      void* workspace, int dtype, hipStream_t st, const BnSums* ready_sums = nullptr);
// ready_sums (may be null): the sums of g and g * xhat are already there (a data-gradient launch
// wrote them, ConvGeom::bnb, and masked dy); they are not computed again, and y must be null.  in_iteration: the launch is one of a
// whole step, beside a weight gradient (bn_shape.h).
hipError_t bn_backward(const void* x, const void* dy, const void* y, const float* gamma,
                       const float* mean, const float* istd, void* dx, float* dgamma, float* dbeta,
                       void* g_out, long rows, int c, void* workspace, int dtype, hipStream_t st,
                       const BnSums* ready_sums = nullptr, bool in_iteration = false);

hipError_t maxpool_forward(const void* x, void* y, int n, int h, int wd, int c, int r, int s,
                           int stride, int pad, int dtype, hipStream_t st);
hipError_t maxpool_backward(const void* x, const void* dy, void* dx, int n, int h, int wd, int c,
                            int r, int s, int stride, int pad, int accumulate, int dtype, hipStream_t st);
hipError_t gap_forward(const void* x, void* y, int n, int hw, int c, int dtype, hipStream_t st);
hipError_t gap_backward(const void* dy, void* dx, int n, int hw, int c, int accumulate, int dtype,
                        hipStream_t st);
// y[row][ch] += b[ch], then max(., 0) if relu
hipError_t bias_add(void* y, const float* b, long rows, int c, int dtype, hipStream_t st, int relu = 0);
// Backward of y = relu(x + b) over rows x c (c % 4 == 0): g = dy * [y > 0] is written over dy (y may
// be null: no mask, dy untouched) and db[ch] = sum over the rows of g (fixed order).
// workspace: relu_bias_workspace_bytes(c) bytes.
size_t relu_bias_workspace_bytes(int c);
// dy[i] = y[i] > 0 ? dy[i] : 0, in place
hipError_t relu_mask(void* dy, const void* y, size_t count, int dtype, hipStream_t st);
hipError_t relu_bias_backward(void* dy, const void* y, float* db, long rows, int c, void* workspace, int dtype,
                              hipStream_t st);
hipError_t column_sum(const void* dy, float* db, long rows, int c, int dtype, hipStream_t st);
// loss_rows: n floats of scratch; loss: one float.  Loss (loss_rows may be null: not wanted) and gradient (dz may be null) in one launch,
// or one of them.
hipError_t softmax_ce(const void* z, const int32_t* labels, float* loss_rows, float* loss, void* dz, int n, int classes, int dtype,
                      hipStream_t st);
hipError_t softmax_ce_forward(const void* z, const int32_t* labels, float* loss_rows, float* loss,
                              int n, int classes, int dtype, hipStream_t st);
hipError_t softmax_ce_backward(const void* z, const int32_t* labels, void* dz, int n, int classes,
                               int dtype, hipStream_t st);
// w <- w - lr * g (fp32); w_bf16 (may be null): rounded copy of the updated weights
hipError_t sgd_update(float* w, const float* g, float lr, size_t count, void* w_bf16, hipStream_t st);
hipError_t fill_zero(float* p, size_t count, hipStream_t st);
// y[n][hw][c] (dtype) = x[n][c][hw] (fp32)
hipError_t nchw_to_nhwc(const float* x, void* y, int n, int c, int hw, int dtype, hipStream_t st);

// Text that acc_last_error(NULL) returns on this thread (calls that have no context).
void set_thread_error(const char* text);

}  // namespace acc
