// Batch normalisation with minibatch statistics over an NHWC tensor viewed as
// rows x c, fused with ReLU and with the residual add of a bottleneck block.
//
// The work is bandwidth bound, so every kernel reads whole float4 channel groups of
// consecutive rows (a wave covers 1 KiB of contiguous memory per load).  Reductions
// over rows run in two fixed-order stages (per-slab partials in double, then a
// workgroup adds the slabs of eight channels in a fixed order): no atomics, results do
// not depend on timing or addresses.
//
// workspace layout (bn_workspace_bytes): double part[2][MAX_SLABS][c] | float coef[4][c]
// (partial sums a convolution launch hands over instead are floats: fp32 sums over 32 rows each)
#include "kernels.h"
#include "dtype.h"

namespace acc {
namespace {

constexpr int MAX_SLABS = kBnMaxSlabs;   // row slabs of the reduction grid (upper bound)
constexpr int THREADS = kBnThreads;
// The finishing kernels: a workgroup adds up FIN_CH channels, FIN_LANES slabs at a time.  The slabs come from memory in
// 64-byte pieces (doubles), every load of a thread in flight at once, so the launch lasts little longer than one trip
// (up to 1024 slabs of 64 to 512 channels, in a step: 9.4 -> 5.9 us against one wave per channel, which used 32 bytes of a line).
constexpr int FIN_CH = 8, FIN_LANES = 128, FIN_THREADS = FIN_CH * FIN_LANES;

// One 16-byte access per thread: four fp32 or eight bf16 channels; or four bf16 channels (8 bytes).
template <class T, int V> struct ElemV;
template <class T> struct ElemV<T, 4> {
  static __device__ __forceinline__ void load(const T* p, float (&v)[4]) { Elem<T>::load4(p, v); }
  static __device__ __forceinline__ void store(T* p, const float (&v)[4]) { Elem<T>::store4(p, v); }
};
template <> struct ElemV<bf16_t, 8> {
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) {
    const uint4 q = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)float_to_bf16(v[2 * i]) | ((uint32_t)float_to_bf16(v[2 * i + 1]) << 16);
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
  }
};

// A tensor, how a workgroup covers its channels, and the rows of one workgroup (0: trips in turn).
struct Span {
  long rows;
  int c, tpr, rpi;
  long rows_per_wg;
};

// Sums over the rows of one slab, per channel, of up to two quantities.  Bound by memory: x (and dy, y) read once, V channels
// = 16 bytes per thread and load, U rows in flight.  With the apply passes below, bf16 512 channels, 256 images of 28x28, residual:
// forward 196 -> 153 us, backward 354 -> 313 (8-byte loads, coefficients fetched per element before); what is left of
// the way to 134 / 223 us of traffic at 4.6 TB/s is the second read: of x, and of dy and y or, where the sums have stored it
// (G; 313 -> 272 us), of the masked gradient, which the caches don't hold.  In slices of 1/2 or 1/4 of the channels, one after the other,
// the rows become too short (862 us both ways), and walking back from the end in the second pass gives nothing.
// The rows of a slab: consecutive ones, or, in a forward pass that reads bf16 eight channels at a time and in a backward pass that stores
// the masked gradient, trips of a few rows dealt out to the slabs in turn, so that the launch as a whole walks through one contiguous window
// after the other (bf16 1024 channels, 81648 rows forward 96.4 -> 90.7 us; fp32 sums alone gain nothing, small ones lose 3 %).
// MODE 0: (x, x*x).   MODE 1: (g, g*xhat) with g = dy * [y > 0] (y optional).
// G: MODE 1 with y, and g is stored (over dy if the caller says so).
template <int MODE, class T, int V, bool G>
__global__ __launch_bounds__(THREADS) void bn_reduce_kernel(const T* __restrict__ x, const T* dy,
                                                            const T* __restrict__ y,
                                                            const float* __restrict__ mean,
                                                            const float* __restrict__ istd,
                                                            double* __restrict__ part, T* g_out, Span sp) {
  __shared__ double red[2][THREADS][V];
  const int tid = threadIdx.x;
  const int lane_r = tid / sp.tpr;            // which row of the iteration
  const int lane_c = tid - lane_r * sp.tpr;   // which channel group
  const int ch = (blockIdx.y * sp.tpr + lane_c) * V;
  const bool active = lane_r < sp.rpi && ch < sp.c;
  const int c = sp.c, rpi = sp.rpi;

  double s0[V], s1[V];
#pragma unroll
  for (int j = 0; j < V; ++j) s0[j] = s1[j] = 0.0;
  if (active) {
    float mu[V], is[V];
    if (MODE == 1) {
#pragma unroll
      for (int j = 0; j < V; ++j) { mu[j] = mean[ch + j]; is[j] = istd[ch + j]; }
    }
    auto add_row = [&](const float (&xs)[V], float (&gv)[V], const float (&ys)[V]) {
      if (MODE == 0) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const double d = (double)xs[j];
          s0[j] += d;
          s1[j] += d * d;
        }
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) {
          gv[j] = !y || ys[j] > 0.f ? gv[j] : 0.f;
          const double gd = (double)gv[j];
          s0[j] += gd;
          s1[j] += gd * (double)((xs[j] - mu[j]) * is[j]);
        }
      }
    };
    // several rows per trip: all their loads are issued before the first sum needs one
    constexpr int U = V == 8 && MODE == 1 ? 2 : 4;
    const bool turns = sp.rows_per_wg == 0;
    const long trip = (long)rpi * U, step = turns ? trip * gridDim.x : trip;
    const long r_lo = (turns ? trip : sp.rows_per_wg) * blockIdx.x + lane_r;
    const long r_hi = turns || r_lo - lane_r + sp.rows_per_wg > sp.rows ? sp.rows : r_lo - lane_r + sp.rows_per_wg;
    if constexpr (!G) {
      const T* px = x + (size_t)r_lo * c + ch;
      const T* pd = MODE == 1 ? dy + (size_t)r_lo * c + ch : nullptr;
      const T* py = MODE == 1 && y ? y + (size_t)r_lo * c + ch : nullptr;
      const size_t hop = (size_t)rpi * c, leap = (size_t)step * c;
      long r = r_lo;
      for (; r + (long)(U - 1) * rpi < r_hi; r += step) {
        float xv[U][V], gv[U][V], yv[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ElemV<T, V>::load(px + u * hop, xv[u]);
          if (MODE == 1) ElemV<T, V>::load(pd + u * hop, gv[u]);
          if (MODE == 1 && y) ElemV<T, V>::load(py + u * hop, yv[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) add_row(xv[u], gv[u], yv[u]);
        px += leap;
        if (MODE == 1) pd += leap;
        if (MODE == 1 && y) py += leap;
      }
      for (; r < r_hi; r += rpi) {                  // rows of the last trip, fewer than U
        float xv[V], gv[V], yv[V];
        ElemV<T, V>::load(px, xv);
        if (MODE == 1) ElemV<T, V>::load(pd, gv);
        if (MODE == 1 && y) ElemV<T, V>::load(py, yv);
        add_row(xv, gv, yv);
        px += hop;
        if (MODE == 1) pd += hop;
        if (MODE == 1 && y) py += hop;
      }
    } else {
      for (long r0 = r_lo; r0 < r_hi; r0 += step) {
        float xv[U][V], gv[U][V], yv[U][V];
        size_t at[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {               // a row that does not exist reads row 0
          const long r = r0 + (long)u * rpi;
          ok[u] = r < r_hi;
          at[u] = (size_t)(ok[u] ? r : 0) * c + ch;
          ElemV<T, V>::load(x + at[u], xv[u]);
          ElemV<T, V>::load(dy + at[u], gv[u]);
          ElemV<T, V>::load(y + at[u], yv[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!ok[u]) break;                        // the rows of a trip go up
          add_row(xv[u], gv[u], yv[u]);
          ElemV<T, V>::store(g_out + at[u], gv[u]);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < V; ++j) {
    red[0][tid][j] = s0[j];
    red[1][tid][j] = s1[j];
  }
  __syncthreads();
  // the first row of threads adds the other rows in order
  if (lane_r == 0 && active) {
    for (int rr = 1; rr < rpi; ++rr) {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        s0[j] += red[0][rr * sp.tpr + lane_c][j];
        s1[j] += red[1][rr * sp.tpr + lane_c][j];
      }
    }
    double* p0 = part + ((size_t)0 * MAX_SLABS + blockIdx.x) * c + ch;
    double* p1 = part + ((size_t)1 * MAX_SLABS + blockIdx.x) * c + ch;
#pragma unroll
    for (int j = 0; j < V; ++j) {
      p0[j] = s0[j];
      p1[j] = s1[j];
    }
  }
}

// out[q][j] = sum over the slabs of part[q][slab][ch0 + j], in a fixed order: thread (l, j) adds slabs l, l + FIN_LANES, ...,
// a butterfly adds the eight l of a wave, and one thread per sum adds the waves.
template <class P>
__device__ __forceinline__ void sum_partials(const P* __restrict__ part, int c, int slabs, int stride, double (&out)[2][FIN_CH]) {
  __shared__ double waves[2][FIN_THREADS / 64][FIN_CH];
  constexpr int PER_LANE = MAX_SLABS / FIN_LANES;
  const int j = threadIdx.x % FIN_CH, l = threadIdx.x / FIN_CH, ch = blockIdx.x * FIN_CH + j;
  P v0[PER_LANE], v1[PER_LANE];
  const P* p0 = part + (ch < c ? ch : 0);
  const P* p1 = p0 + (size_t)stride * c;      // part[2][stride][c]
#pragma unroll
  for (int u = 0; u < PER_LANE; ++u) {
    const int k = l + FIN_LANES * u;
    const size_t at = k < slabs ? (size_t)k * c : 0;   // slab 0 always exists; its value is dropped
    v0[u] = p0[at];
    v1[u] = p1[at];
  }
  double a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int u = 0; u < PER_LANE; ++u) {
    const bool ok = l + FIN_LANES * u < slabs;
    a0 += ok ? (double)v0[u] : 0.0;
    a1 += ok ? (double)v1[u] : 0.0;
  }
#pragma unroll
  for (int o = FIN_CH; o < 64; o <<= 1) { a0 += __shfl_xor(a0, o); a1 += __shfl_xor(a1, o); }
  if ((threadIdx.x & 63) < FIN_CH) {
    waves[0][threadIdx.x / 64][j] = a0;
    waves[1][threadIdx.x / 64][j] = a1;
  }
  __syncthreads();
  if (threadIdx.x < 2 * FIN_CH) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < FIN_THREADS / 64; ++w) t += waves[threadIdx.x / FIN_CH][w][j];
    out[threadIdx.x / FIN_CH][j] = t;
  }
  __syncthreads();
}

// forward:  mean, istd; coef[0] = scale = gamma*istd, coef[1] = mean, coef[2] = beta
template <class P>
__global__ __launch_bounds__(FIN_THREADS) void bn_fwd_finish_kernel(
    const P* __restrict__ part, const float* __restrict__ gamma, const float* __restrict__ beta,
    float* __restrict__ mean, float* __restrict__ istd, float* __restrict__ coef, long rows, int c,
    float eps, int slabs, int stride) {
  const int j = threadIdx.x % FIN_CH, ch = blockIdx.x * FIN_CH + j;
  // the channel's parameters are fetched beside the partial sums, not after them
  const float gam = gamma[ch < c ? ch : 0], bet = beta[ch < c ? ch : 0];
  __shared__ double out[2][FIN_CH];
  sum_partials(part, c, slabs, stride, out);
  if (threadIdx.x >= FIN_CH || ch >= c) return;
  const double sum = out[0][j], ss = out[1][j];
  const double m = (double)rows;
  const double mu = sum / m;
  double var = ss / m - mu * mu;
  if (var < 0.0) var = 0.0;
  const double is = 1.0 / sqrt(var + (double)eps);
  mean[ch] = (float)mu;
  istd[ch] = (float)is;
  const double scale = (double)gam * is;
  coef[ch] = (float)scale;
  coef[c + ch] = (float)mu;
  coef[2 * c + ch] = bet;
}

// backward: dbeta, dgamma; coef[0] = a = gamma*istd, coef[1] = dbeta/m, coef[2] = dgamma/m
template <class P>
__global__ __launch_bounds__(FIN_THREADS) void bn_bwd_finish_kernel(
    const P* __restrict__ part, const float* __restrict__ gamma, const float* __restrict__ istd,
    float* __restrict__ dgamma, float* __restrict__ dbeta, float* __restrict__ coef, long rows, int c,
    int slabs, int stride) {
  const int j = threadIdx.x % FIN_CH, ch = blockIdx.x * FIN_CH + j;
  const float gam = gamma[ch < c ? ch : 0], is = istd[ch < c ? ch : 0];
  __shared__ double out[2][FIN_CH];
  sum_partials(part, c, slabs, stride, out);
  if (threadIdx.x >= FIN_CH || ch >= c) return;
  const double db = out[0][j], dg = out[1][j];
  dbeta[ch] = (float)db;
  dgamma[ch] = (float)dg;
  const double m = (double)rows;
  coef[ch] = gam * is;
  coef[c + ch] = (float)(db / m);
  coef[2 * c + ch] = (float)(dg / m);
}

// The apply passes: the groups of V channels of the tensor in memory order, thread i of the first `stride` taking groups i,
// i + stride, ...; stride is a multiple of the groups of a row, so a thread keeps its channels (`tpc` groups a row), the
// coefficients stay in registers and the launch as a whole reads and writes one contiguous window after the other,
// whatever the channel count.  bf16, both directions (coefficients fetched per element / a workgroup walking down rows of its
// own, four or two in flight / so): 512 channels, 256 images of 28x28, residual 550 / 482 / 466 us; 760, 38 of 51x51,
// residual 416 / 427 / 343; 1028, 41 of 28x28 133 / 148 / 124.  Several loads of a thread in flight gain nothing here (four: 491, 349, 129).
struct Flat {
  size_t groups, stride;
  int c, tpc;
};

// y = relu?((x-mean)*scale + beta (+ res)).  Subtracting the mean first keeps the result exact where x equals the mean (a channel
// of constant values).
template <class T, int V>
__global__ __launch_bounds__(THREADS) void bn_apply_kernel(const T* __restrict__ x,
                                                           const T* __restrict__ res,
                                                           const float* __restrict__ coef,
                                                           T* __restrict__ y, int relu, Flat fl) {
  const size_t i0 = (size_t)blockIdx.x * THREADS + threadIdx.x;
  if (i0 >= fl.stride) return;
  const int c = fl.c, ch = (int)(i0 % fl.tpc) * V;
  float sc[V], mu[V], be[V];
#pragma unroll
  for (int j = 0; j < V; ++j) { sc[j] = coef[ch + j]; mu[j] = coef[c + ch + j]; be[j] = coef[2 * c + ch + j]; }
  const size_t hop = fl.stride * V, end = fl.groups * V;
  for (size_t at = i0 * V; at < end; at += hop) {
    float xv[V], rv[V], o[V];
    ElemV<T, V>::load(x + at, xv);
    if (res) ElemV<T, V>::load(res + at, rv);
#pragma unroll
    for (int j = 0; j < V; ++j) {
      o[j] = fmaf(xv[j] - mu[j], sc[j], be[j]);
      if (res) o[j] += rv[j];
      if (relu) o[j] = fmaxf(o[j], 0.f);
    }
    ElemV<T, V>::store(y + at, o);
  }
}

// dx = a*(g - dbeta/m - xhat*dgamma/m), g = dy*[y>0]; optionally stores g (may alias dy)
template <class T, int V>
__global__ __launch_bounds__(THREADS) void bn_bwd_apply_kernel(
    const T* __restrict__ x, const T* dy, const T* __restrict__ y,
    const float* __restrict__ mean, const float* __restrict__ istd, const float* __restrict__ coef,
    T* __restrict__ dx, T* g_out, Flat fl) {
  const size_t i0 = (size_t)blockIdx.x * THREADS + threadIdx.x;
  if (i0 >= fl.stride) return;
  const int c = fl.c, ch = (int)(i0 % fl.tpc) * V;
  float mu[V], is[V], a[V], c1[V], c2[V];
#pragma unroll
  for (int j = 0; j < V; ++j) {
    mu[j] = mean[ch + j]; is[j] = istd[ch + j];
    a[j] = coef[ch + j]; c1[j] = coef[c + ch + j]; c2[j] = coef[2 * c + ch + j];
  }
  const size_t hop = fl.stride * V, end = fl.groups * V;
  for (size_t at = i0 * V; at < end; at += hop) {
    float xv[V], gv[V], yv[V], o[V];
    ElemV<T, V>::load(x + at, xv);
    ElemV<T, V>::load(dy + at, gv);
    if (y) ElemV<T, V>::load(y + at, yv);
#pragma unroll
    for (int j = 0; j < V; ++j) {
      gv[j] = !y || yv[j] > 0.f ? gv[j] : 0.f;
      o[j] = a[j] * (gv[j] - c1[j] - (xv[j] - mu[j]) * is[j] * c2[j]);
    }
    ElemV<T, V>::store(dx + at, o);
    if (g_out) ElemV<T, V>::store(g_out + at, gv);
  }
}

// ---- finish + apply in one launch, for reductions with few slabs
//
// The finishing kernels above are two dependent trips to memory and a launch of their own
// between the sums and the apply pass.  Where the sums come in few slabs, every workgroup of
// the apply pass adds the slabs of its own 32 channels itself (same order in every workgroup,
// so all of them arrive at the same coefficients) while its first rows are on their way, one
// thread per channel works out the coefficients, and the workgroups of the first row slab
// also store the per-channel results.  A workgroup covers a column slice of 32 channels
// (8 threads x 4 channels across a row) and 32 rows per trip, four trips in flight.
constexpr int SL_TPR = 8;                   // threads across the 32 channels of a slice
constexpr int SL_CH = SL_TPR * 4;
constexpr int SL_ROWS = THREADS / SL_TPR;   // rows per trip
constexpr int SL_BATCH = 16;                // 16-byte partial loads a thread has in flight
constexpr int SL_U = 4;                     // rows of a thread in flight in the apply loop
constexpr int SL_WGS = 256;                 // workgroups of a launch, about: one per CU.  Every workgroup re-reads its
                                            // slice's partials, and in the step the kernel shares the chip with a weight
                                            // gradient (ResNet-152 at minibatch 41, images/s at 192 / 256 / 320 / 384 /
                                            // 512 / 768 / 1024: 1215 / 1233 / 1216 / 1218 / 1223 / 1219 / 1218)
constexpr int kSlicePhasesMax = 16;

struct SliceScratch {
  double red[2][kSlicePhasesMax][SL_CH];
  double tot[2][SL_CH];
  float coef[3][SL_CH];
};

// tot[q][j] = sum over the slabs of part[q][slab][ch0 + j].  A 16-byte load covers VEC
// neighbouring channels of one slab; thread (col, plane, phase) adds the slabs phase,
// phase + PHASES, ... of its channels, then 64 threads add the phases in order.
template <class P>
__device__ __forceinline__ void slice_sums(const P* __restrict__ part, int c, int slabs, int stride, int ch0,
                                           SliceScratch& sh) {
  constexpr int VEC = 16 / sizeof(P), COLS = SL_CH / VEC, PHASES = THREADS / (2 * COLS);
  static_assert(PHASES <= kSlicePhasesMax, "scratch");
  struct alignas(16) Vec { P v[VEC]; };
  const int tid = threadIdx.x;
  const int col = tid % COLS, plane = (tid / COLS) & 1, phase = tid / (2 * COLS);
  const int ch = ch0 + col * VEC;
  const bool ch_ok = ch < c;                // c is a multiple of 4: the VEC channels exist together
  const P* p = part + (size_t)plane * stride * c + (ch_ok ? ch : 0);
  double a[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) a[j] = 0.0;
  for (int base = 0; base < slabs; base += PHASES * SL_BATCH) {
    Vec v[SL_BATCH];
#pragma unroll
    for (int u = 0; u < SL_BATCH; ++u) {
      const int k = base + phase + PHASES * u;
      v[u] = *reinterpret_cast<const Vec*>(p + (k < slabs ? (size_t)k * c : 0));   // slab 0 always exists
    }
#pragma unroll
    for (int u = 0; u < SL_BATCH; ++u) {
      const bool ok = ch_ok && base + phase + PHASES * u < slabs;
#pragma unroll
      for (int j = 0; j < VEC; ++j) a[j] += ok ? (double)v[u].v[j] : 0.0;
    }
  }
#pragma unroll
  for (int j = 0; j < VEC; ++j) sh.red[plane][phase][col * VEC + j] = a[j];
  __syncthreads();
  if (tid < 2 * SL_CH) {
    const int q = tid / SL_CH, j = tid % SL_CH;
    double t = 0.0;
#pragma unroll
    for (int ph = 0; ph < PHASES; ++ph) t += sh.red[q][ph][j];
    sh.tot[q][j] = t;
  }
  __syncthreads();
}

template <class T, class P>
__global__ __launch_bounds__(THREADS) void bn_fwd_slice_kernel(
    const T* __restrict__ x, const T* __restrict__ res, const P* __restrict__ part,
    const float* __restrict__ gamma, const float* __restrict__ beta, float* __restrict__ mean,
    float* __restrict__ istd, T* __restrict__ y, long rows, int c, int relu, float eps, int slabs, int stride,
    long rows_per_wg) {
  __shared__ SliceScratch sh;
  const int ch0 = blockIdx.y * SL_CH;
  const int lane_c = threadIdx.x % SL_TPR, lane_r = threadIdx.x / SL_TPR;
  const int ch = ch0 + lane_c * 4;
  const bool active = ch < c;
  float bet[4] = {0, 0, 0, 0};
  if (active) {
    const float4 b4 = *reinterpret_cast<const float4*>(beta + ch);
    bet[0] = b4.x; bet[1] = b4.y; bet[2] = b4.z; bet[3] = b4.w;
  }
  const long r_lo = (long)blockIdx.x * rows_per_wg;
  const long r_hi = r_lo + rows_per_wg < rows ? r_lo + rows_per_wg : rows;
  float xv[SL_U][4], rv[SL_U][4] = {};
  auto load_trip = [&](long r) {
#pragma unroll
    for (int u = 0; u < SL_U; ++u) {
      const long ru = r + (long)u * SL_ROWS;
      if (active && ru < r_hi) {
        const size_t off = (size_t)ru * c + ch;
        Elem<T>::load4(x + off, xv[u]);
        if (res) Elem<T>::load4(res + off, rv[u]);
      }
    }
  };
  load_trip(r_lo + lane_r);   // requested before the sums, so that they travel meanwhile
  slice_sums(part, c, slabs, stride, ch0, sh);
  if (threadIdx.x < SL_CH && ch0 + threadIdx.x < c) {
    const int j = threadIdx.x;
    const double m = (double)rows;
    const double mean_d = sh.tot[0][j] / m;
    double var = sh.tot[1][j] / m - mean_d * mean_d;
    if (var < 0.0) var = 0.0;
    const double is_d = 1.0 / sqrt(var + (double)eps);
    sh.coef[0][j] = (float)mean_d;
    sh.coef[1][j] = (float)((double)gamma[ch0 + j] * is_d);
    if (blockIdx.x == 0) {
      mean[ch0 + j] = (float)mean_d;
      istd[ch0 + j] = (float)is_d;
    }
  }
  __syncthreads();
  if (!active) return;
  float mu[4], sc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    mu[j] = sh.coef[0][lane_c * 4 + j];
    sc[j] = sh.coef[1][lane_c * 4 + j];
  }
  for (long r = r_lo + lane_r; r < r_hi; r += (long)SL_U * SL_ROWS) {
    if (r != r_lo + lane_r) load_trip(r);
#pragma unroll
    for (int u = 0; u < SL_U; ++u) {
      const long ru = r + (long)u * SL_ROWS;
      if (ru < r_hi) {
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          o[j] = fmaf(xv[u][j] - mu[j], sc[j], bet[j]);
          if (res) o[j] += rv[u][j];
          if (relu) o[j] = fmaxf(o[j], 0.f);
        }
        Elem<T>::store4(y + (size_t)ru * c + ch, o);
      }
    }
  }
}

template <class T, class P>
__global__ __launch_bounds__(THREADS) void bn_bwd_slice_kernel(
    const T* __restrict__ x, const T* dy, const T* __restrict__ y, const P* __restrict__ part,
    const float* __restrict__ gamma, const float* __restrict__ mean, const float* __restrict__ istd,
    float* __restrict__ dgamma, float* __restrict__ dbeta, T* __restrict__ dx, T* g_out, long rows, int c,
    int slabs, int stride, long rows_per_wg) {
  __shared__ SliceScratch sh;
  const int ch0 = blockIdx.y * SL_CH;
  const int lane_c = threadIdx.x % SL_TPR, lane_r = threadIdx.x / SL_TPR;
  const int ch = ch0 + lane_c * 4;
  const bool active = ch < c;
  float a[4] = {0, 0, 0, 0}, mu[4] = {0, 0, 0, 0}, is[4] = {0, 0, 0, 0};
  if (active) {
    const float4 g4 = *reinterpret_cast<const float4*>(gamma + ch);
    const float4 m4 = *reinterpret_cast<const float4*>(mean + ch);
    const float4 i4 = *reinterpret_cast<const float4*>(istd + ch);
    mu[0] = m4.x; mu[1] = m4.y; mu[2] = m4.z; mu[3] = m4.w;
    is[0] = i4.x; is[1] = i4.y; is[2] = i4.z; is[3] = i4.w;
    a[0] = g4.x * i4.x; a[1] = g4.y * i4.y; a[2] = g4.z * i4.z; a[3] = g4.w * i4.w;
  }
  const long r_lo = (long)blockIdx.x * rows_per_wg;
  const long r_hi = r_lo + rows_per_wg < rows ? r_lo + rows_per_wg : rows;
  float xv[SL_U][4], gv[SL_U][4], yv[SL_U][4] = {};
  auto load_trip = [&](long r) {
#pragma unroll
    for (int u = 0; u < SL_U; ++u) {
      const long ru = r + (long)u * SL_ROWS;
      if (active && ru < r_hi) {
        const size_t off = (size_t)ru * c + ch;
        Elem<T>::load4(x + off, xv[u]);
        Elem<T>::load4(dy + off, gv[u]);
        if (y) Elem<T>::load4(y + off, yv[u]);
      }
    }
  };
  load_trip(r_lo + lane_r);
  slice_sums(part, c, slabs, stride, ch0, sh);
  if (threadIdx.x < SL_CH && ch0 + threadIdx.x < c) {
    const int j = threadIdx.x;
    const double m = (double)rows;
    const double db_d = sh.tot[0][j], dg_d = sh.tot[1][j];
    sh.coef[0][j] = (float)(db_d / m);
    sh.coef[1][j] = (float)(dg_d / m);
    if (blockIdx.x == 0) {
      dbeta[ch0 + j] = (float)db_d;
      dgamma[ch0 + j] = (float)dg_d;
    }
  }
  __syncthreads();
  if (!active) return;
  float c1[4], c2[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    c1[j] = sh.coef[0][lane_c * 4 + j];
    c2[j] = sh.coef[1][lane_c * 4 + j];
  }
  for (long r = r_lo + lane_r; r < r_hi; r += (long)SL_U * SL_ROWS) {
    if (r != r_lo + lane_r) load_trip(r);
#pragma unroll
    for (int u = 0; u < SL_U; ++u) {
      const long ru = r + (long)u * SL_ROWS;
      if (ru < r_hi) {
        float o[4], g[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          g[j] = (!y || yv[u][j] > 0.f) ? gv[u][j] : 0.f;
          o[j] = a[j] * (g[j] - c1[j] - (xv[u][j] - mu[j]) * is[j] * c2[j]);
        }
        const size_t off = (size_t)ru * c + ch;
        Elem<T>::store4(dx + off, o);
        if (g_out) Elem<T>::store4(g_out + off, g);
      }
    }
  }
}

// grid of the slice kernels: about SL_WGS workgroups over all column slices, a whole number of
// SL_U-row trips per workgroup; a function of the shape only
inline dim3 slice_grid(long rows, int c, long* rows_per_wg) {
  const int slices = (c + SL_CH - 1) / SL_CH;
  const long slabs = SL_WGS / slices > 0 ? SL_WGS / slices : 1;
  const long trip = (long)SL_U * SL_ROWS;
  long per = (rows + slabs - 1) / slabs;
  per = (per + trip - 1) / trip * trip;
  *rows_per_wg = per;
  return dim3((unsigned)((rows + per - 1) / per), (unsigned)slices);
}

// about 16 workgroups per compute unit at most, and threads for a whole number of rows
inline Flat apply_flat(long rows, int c, int v, unsigned* blocks) {
  Flat f{(size_t)rows * (c / v), 0, c, c / v};
  const size_t want = (f.groups + THREADS - 1) / THREADS, cap = 256 * 16;
  size_t b = want < cap ? want : cap;
  if (b * THREADS < (size_t)f.tpc) b = ((size_t)f.tpc + THREADS - 1) / THREADS;      // at least one row
  f.stride = b * THREADS / f.tpc * f.tpc;
  *blocks = (unsigned)b;
  return f;
}

}  // namespace

size_t bn_workspace_bytes(int c) {
  return (size_t)2 * MAX_SLABS * c * sizeof(double) + (size_t)4 * c * sizeof(float);
}

namespace {

// finish + apply of the forward pass from `slabs` partial sums of type P
template <class T, int V, class P>
void bn_forward_finish(const T* x, const float* gamma, const float* beta, const T* res, T* y, float* mean, float* istd,
                       long rows, int c, int relu, float eps, const P* sums, int slabs, int stride,
                       float* coef, hipStream_t st) {
  hipLaunchKernelGGL(bn_fwd_finish_kernel<P>, dim3((c + FIN_CH - 1) / FIN_CH), dim3(FIN_THREADS), 0, st, sums, gamma,
                     beta, mean, istd, coef, rows, c, eps, slabs, stride);
  unsigned blocks;
  const Flat fl = apply_flat(rows, c, V, &blocks);
  hipLaunchKernelGGL((bn_apply_kernel<T, V>), dim3(blocks), dim3(THREADS), 0, st, x, res, coef, y, relu, fl);
}

template <class T, class P>
void bn_forward_slices(const T* x, const float* gamma, const float* beta, const T* res, T* y, float* mean, float* istd,
                       long rows, int c, int relu, float eps, const P* sums, int slabs, int stride, hipStream_t st) {
  long per;
  const dim3 grid = slice_grid(rows, c, &per);
  hipLaunchKernelGGL((bn_fwd_slice_kernel<T, P>), grid, dim3(THREADS), 0, st, x, res, sums, gamma, beta, mean, istd,
                     y, rows, c, relu, eps, slabs, stride, per);
}

template <class T, int V>
hipError_t bn_forward_v(const T* x, const float* gamma, const float* beta, const T* res, T* y, float* mean,
                        float* istd, long rows, int c, int relu, float eps, void* workspace, hipStream_t st,
                        const BnSums& ready) {
  double* part = static_cast<double*>(workspace);
  float* coef = reinterpret_cast<float*>(part + (size_t)2 * MAX_SLABS * c);
  if (ready.part) {   // the producer of x left the sums
    if (slice_takes((int)sizeof(T), rows, ready.slabs))
      bn_forward_slices(x, gamma, beta, res, y, mean, istd, rows, c, relu, eps, ready.part, ready.slabs, ready.stride, st);
    else
      bn_forward_finish<T, V>(x, gamma, beta, res, y, mean, istd, rows, c, relu, eps, ready.part, ready.slabs, ready.stride,
                              coef, st);
    return hipGetLastError();
  }
  const SumShape rs = bn_sum_shape(rows, c, V, (int)sizeof(T), /*backward=*/false, /*stores=*/false);
  const int slabs = rs.slabs;
  hipLaunchKernelGGL((bn_reduce_kernel<0, T, V, false>), dim3(slabs, rs.col_slices), dim3(THREADS), 0, st, x, (const T*)nullptr,
                     (const T*)nullptr, nullptr, nullptr, part, (T*)nullptr, Span{rows, c, rs.tpr, rs.rpi, V == 8 ? 0 : (rows + slabs - 1) / slabs});
  if (slice_takes((int)sizeof(T), rows, rs.slabs))
    bn_forward_slices(x, gamma, beta, res, y, mean, istd, rows, c, relu, eps, (const double*)part, slabs, MAX_SLABS, st);
  else
    bn_forward_finish<T, V>(x, gamma, beta, res, y, mean, istd, rows, c, relu, eps, (const double*)part, slabs, MAX_SLABS, coef, st);
  return hipGetLastError();
}

template <class T, int V, class P>
void bn_backward_finish(const T* x, const T* dy, const T* y, const float* gamma, const float* mean, const float* istd,
                        T* dx, float* dgamma, float* dbeta, T* g_out, long rows, int c, const P* sums, int slabs,
                        int stride, float* coef, hipStream_t st) {
  hipLaunchKernelGGL(bn_bwd_finish_kernel<P>, dim3((c + FIN_CH - 1) / FIN_CH), dim3(FIN_THREADS), 0, st, sums, gamma,
                     istd, dgamma, dbeta, coef, rows, c, slabs, stride);
  unsigned blocks;
  const Flat fl = apply_flat(rows, c, V, &blocks);
  hipLaunchKernelGGL((bn_bwd_apply_kernel<T, V>), dim3(blocks), dim3(THREADS), 0, st, x, dy, y, mean, istd, coef, dx, g_out, fl);
}

template <class T, class P>
void bn_backward_slices(const T* x, const T* dy, const T* y, const float* gamma, const float* mean, const float* istd,
                        T* dx, float* dgamma, float* dbeta, T* g_out, long rows, int c, const P* sums, int slabs,
                        int stride, hipStream_t st) {
  long per;
  const dim3 grid = slice_grid(rows, c, &per);
  hipLaunchKernelGGL((bn_bwd_slice_kernel<T, P>), grid, dim3(THREADS), 0, st, x, dy, y, sums, gamma, mean, istd,
                     dgamma, dbeta, dx, g_out, rows, c, slabs, stride, per);
}

template <class T, int V>
hipError_t bn_backward_v(const T* x, const T* dy, const T* y, const float* gamma, const float* mean,
                         const float* istd, T* dx, float* dgamma, float* dbeta, T* g_out, long rows, int c,
                         void* workspace, hipStream_t st, const BnSums& ready, bool in_iteration) {
  double* part = static_cast<double*>(workspace);
  float* coef = reinterpret_cast<float*>(part + (size_t)2 * MAX_SLABS * c);
  if (ready.part) {   // the data gradient left the sums
    if (slice_takes((int)sizeof(T), rows, ready.slabs))
      bn_backward_slices(x, dy, y, gamma, mean, istd, dx, dgamma, dbeta, g_out, rows, c, ready.part, ready.slabs, ready.stride, st);
    else
      bn_backward_finish<T, V>(x, dy, y, gamma, mean, istd, dx, dgamma, dbeta, g_out, rows, c, ready.part, ready.slabs,
                               ready.stride, coef, st);
    return hipGetLastError();
  }
  // (not over x, which the next pass reads)
  const bool g_early = y && g_out && g_out != x && bn_stores_early(rows, c, (int)sizeof(T), in_iteration);
  const SumShape rs = bn_sum_shape(rows, c, V, (int)sizeof(T), /*backward=*/true, g_early);
  const int slabs = rs.slabs;
  if (g_early)
    hipLaunchKernelGGL((bn_reduce_kernel<1, T, V, true>), dim3(slabs, rs.col_slices), dim3(THREADS), 0, st, x, dy, y, mean,
                       istd, part, g_out, Span{rows, c, rs.tpr, rs.rpi, 0});
  else
    hipLaunchKernelGGL((bn_reduce_kernel<1, T, V, false>), dim3(slabs, rs.col_slices), dim3(THREADS), 0, st, x, dy, y, mean,
                       istd, part, (T*)nullptr, Span{rows, c, rs.tpr, rs.rpi, (rows + slabs - 1) / slabs});
  if (g_early) { dy = g_out; y = nullptr; g_out = nullptr; }
  if (slice_takes((int)sizeof(T), rows, rs.slabs))
    bn_backward_slices(x, dy, y, gamma, mean, istd, dx, dgamma, dbeta, g_out, rows, c, (const double*)part, slabs, MAX_SLABS, st);
  else
    bn_backward_finish<T, V>(x, dy, y, gamma, mean, istd, dx, dgamma, dbeta, g_out, rows, c, (const double*)part, slabs,
                             MAX_SLABS, coef, st);
  return hipGetLastError();
}

}  // namespace

// bf16, eight channels per thread: the channels come in eights (every row then starts on a 16-byte address, as every tensor does)
// and there are rows enough for the threads left (512 channels, 256 images of 28x28, both ways 510 us against 556 with four;
// 40 channels, 200 images of 14x14, half the workgroups: 32 against 27; smaller tensors run the slice kernels: 512 channels,
// 49 images of 9x9 31 against 26).
static bool wide_bf16(long rows, int c) { return c % 8 == 0 && rows > kSliceMaxRows && rows * c >= (4L << 20); }

hipError_t bn_forward(const void* x, const float* gamma, const float* beta, const void* res, void* y,
                      float* mean, float* istd, long rows, int c, int relu, float eps, void* workspace,
                      int dtype, hipStream_t st, const BnSums* ready_sums) {
  if (!x || !gamma || !beta || !y || !mean || !istd || !workspace) return hipErrorInvalidValue;
  if (rows <= 0 || c <= 0 || (c & 3)) return hipErrorInvalidValue;
  const BnSums ready = ready_sums ? *ready_sums : BnSums{nullptr, 0, 0};
  if (ready.part && (ready.slabs <= 0 || ready.slabs > MAX_SLABS || ready.stride < ready.slabs)) return hipErrorInvalidValue;
  if (dtype == DT_F32)
    return bn_forward_v<float, 4>((const float*)x, gamma, beta, (const float*)res, (float*)y, mean, istd, rows, c, relu, eps,
                        workspace, st, ready);
  if (dtype == DT_BF16 && wide_bf16(rows, c))
    return bn_forward_v<bf16_t, 8>((const bf16_t*)x, gamma, beta, (const bf16_t*)res, (bf16_t*)y, mean, istd, rows, c, relu,
                                   eps, workspace, st, ready);
  if (dtype == DT_BF16)
    return bn_forward_v<bf16_t, 4>((const bf16_t*)x, gamma, beta, (const bf16_t*)res, (bf16_t*)y, mean, istd, rows, c, relu,
                        eps, workspace, st, ready);
  return hipErrorInvalidValue;
}

hipError_t bn_backward(const void* x, const void* dy, const void* y, const float* gamma, const float* mean,
                       const float* istd, void* dx, float* dgamma, float* dbeta, void* g_out, long rows, int c,
                       void* workspace, int dtype, hipStream_t st, const BnSums* ready_sums, bool in_iteration) {
  if (!x || !dy || !gamma || !mean || !istd || !dx || !dgamma || !dbeta || !workspace)
    return hipErrorInvalidValue;
  if (rows <= 0 || c <= 0 || (c & 3)) return hipErrorInvalidValue;
  const BnSums ready = ready_sums ? *ready_sums : BnSums{nullptr, 0, 0};
  if (ready.part && (y || ready.slabs <= 0 || ready.slabs > MAX_SLABS || ready.stride < ready.slabs))
    return hipErrorInvalidValue;
  if (dtype == DT_F32)
    return bn_backward_v<float, 4>((const float*)x, (const float*)dy, (const float*)y, gamma, mean, istd, (float*)dx, dgamma,
                         dbeta, (float*)g_out, rows, c, workspace, st, ready, in_iteration);
  if (dtype == DT_BF16 && wide_bf16(rows, c))
    return bn_backward_v<bf16_t, 8>((const bf16_t*)x, (const bf16_t*)dy, (const bf16_t*)y, gamma, mean, istd, (bf16_t*)dx,
                                    dgamma, dbeta, (bf16_t*)g_out, rows, c, workspace, st, ready, in_iteration);
  if (dtype == DT_BF16)
    return bn_backward_v<bf16_t, 4>((const bf16_t*)x, (const bf16_t*)dy, (const bf16_t*)y, gamma, mean, istd, (bf16_t*)dx,
                         dgamma, dbeta, (bf16_t*)g_out, rows, c, workspace, st, ready, in_iteration);
  return hipErrorInvalidValue;
}

}  // namespace acc
