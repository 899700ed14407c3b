// fp32 products of few rows and long reductions (a fully connected layer and its data gradient, 1x1 convolutions of a few images):
//
//   out[m][n] (+)= sum_k A[m][k] * W(k, n),     W stored [n][k], or [k][n] as it is before a data gradient's transposition
//
// The tiles of the other kernels leave most of the chip idle here (41 x 1000: sixteen tiles of 64 x 64) and each of them is a chain
// of trips through LDS.  Here a workgroup of sixteen waves owns 16 rows by 16 columns (up to 64 with W[k][n]); the waves deal
// out the values of K, read their fragments straight from memory into registers, several groups ahead, multiply with
// v_mfma_f32_16x16x4_f32, and the workgroup adds their sums up in wave order.  A [k][n] filter is read as it lies: a lane takes
// four columns of one k in 16 bytes, one column per block of the result, so nothing transposes it first.
//
// Bound: a launch's fixed 4 us and a trip to memory or two; with several tiles per compute unit the rows and columns that each of them
// reads again out of the caches.  The layer that ends a ResNet (41 images, 2048 -> 1000): forward 29.2 -> 10.4 us, data gradient 37 -> 7.8.
#include "kernels.h"
#include "dtype.h"
#include "side_wide.h"

namespace acc {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
constexpr int RW_THREADS = 1024, RW_WAVES = 16;

[[maybe_unused]] __device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
#else
  return c;  // the host pass never runs this
#endif
}

// A lane's place in a fragment: row or column lane % 16, the k of its group lane / 16.  CN = 0: W is [n][k], 16 columns, eight k per
// lane in two loads.  CN = 1, 2, 4: W is [k][n], 16 * CN columns, a lane takes four k of A in one load and CN columns of each
// of these k.
template <int CN>
__global__ __launch_bounds__(RW_THREADS, 4) void igemm_rows_kernel(ConvGeom g, int M, int K, int n_tiles_n, int n_tiles, int main_grid) {
  [[maybe_unused]] constexpr bool KN = CN > 0;
  [[maybe_unused]] constexpr int NB = KN ? CN : 1, BN = 16 * NB;      // blocks of 16 columns, columns
  [[maybe_unused]] constexpr int LK = KN ? 4 : 8, GK = 4 * LK;        // values of K per lane, per group
  [[maybe_unused]] constexpr int U = 2;                               // groups per batch of loads; two batches on their way
  [[maybe_unused]] constexpr int NS = NB > 1 ? 2 : 4;                 // sums per block: shorter chains of roundings, and nothing waits for the one before
  constexpr int TILE = 16 * BN;
  __shared__ __attribute__((aligned(16))) float lds[RW_WAVES * TILE];
  if ((int)blockIdx.x >= main_grid) {
    reduce_wide<RW_THREADS>(g.side, (int)blockIdx.x - main_grid);
    return;
  }
#if defined(__HIP_DEVICE_COMPILE__)
  // an XCD's workgroups take neighbouring tiles, all rows of one piece of the filter before the next
  const int tile = (blockIdx.x & 7) * (main_grid >> 3) + (blockIdx.x >> 3);
  if (tile >= n_tiles) return;
  const int tiles_m = n_tiles / n_tiles_n, m0 = (tile % tiles_m) * 16, n0 = (tile / tiles_m) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rc = lane & 15, kg = lane >> 4;
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;                    // beyond any descriptor range: reads as zero
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.in), 0, (int)(uint32_t)((size_t)M * K * 4), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(KN ? g.w_kn : g.w), 0, (int)(uint32_t)((size_t)g.n_out * K * 4), 0x00020000);
  const int groups = (K + GK - 1) / GK, m = m0 + rc, n = n0 + (KN ? CN * rc : rc);
  const bool m_ok = m < M, n_ok = n < g.n_out;                 // columns come in fours
  struct Batch {
    float a[U][LK], b[U][LK][NB];
  };
  auto four = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t at, float& x0, float& x1, float& x2, float& x3) {
    const v4u v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, 0, 0);
    x0 = __uint_as_float(v[0]); x1 = __uint_as_float(v[1]); x2 = __uint_as_float(v[2]); x3 = __uint_as_float(v[3]);
  };
  auto load = [&](Batch& x, int t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (t0 + u * RW_WAVES) * GK + kg * LK;        // the lane's first k; all of its values exist, or none
      const bool k_ok = k < K;
#pragma unroll
      for (int v = 0; v < LK; v += 4)
        four(ra, k_ok && m_ok ? ((uint32_t)m * (uint32_t)K + (uint32_t)(k + v)) * 4u : OUTSIDE, x.a[u][v], x.a[u][v + 1], x.a[u][v + 2], x.a[u][v + 3]);
      if constexpr (!KN) {
#pragma unroll
        for (int v = 0; v < LK; v += 4)
          four(rb, k_ok && n_ok ? ((uint32_t)n * (uint32_t)K + (uint32_t)(k + v)) * 4u : OUTSIDE, x.b[u][v][0], x.b[u][v + 1][0], x.b[u][v + 2][0], x.b[u][v + 3][0]);
      } else {
#pragma unroll
        for (int v = 0; v < LK; ++v) {
          const uint32_t at = k_ok && n_ok ? ((uint32_t)(k + v) * (uint32_t)g.n_out + (uint32_t)n) * 4u : OUTSIDE;
          if constexpr (CN == 4) {
            four(rb, at, x.b[u][v][0], x.b[u][v][1], x.b[u][v][2], x.b[u][v][3]);
          } else if constexpr (CN == 2) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(rb, (int)at, 0, 0);
            x.b[u][v][0] = __uint_as_float(w[0]);
            x.b[u][v][1] = __uint_as_float(w[1]);
          } else {
            x.b[u][v][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (int)at, 0, 0));
          }
        }
      }
    }
  };
  v4f acc[NS][NB];
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const Batch& x) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < LK; ++v)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[v % NS][j] = mfma4(x.a[u][v], x.b[u][v][j], acc[v % NS][j]);
  };
  constexpr int STEP = U * RW_WAVES;
  Batch x0, x1;
  load(x0, wave);
  for (int t = wave; t < groups; t += 2 * STEP) {
    load(x1, t + STEP);                                        // a batch beyond K reads nothing
    multiply(x0);
    if (t + STEP >= groups) break;
    load(x0, t + 2 * STEP);
    multiply(x1);
  }
  // ---- the waves' sums through LDS, [wave][row][column], added in wave order
#pragma unroll
  for (int j = 0; j < NB; ++j) {
#pragma unroll
    for (int d = NS / 2; d > 0; d /= 2)
#pragma unroll
      for (int i = 0; i < d; ++i) acc[i][j] += acc[i + d][j];
#pragma unroll
    for (int v = 0; v < 4; ++v) lds[wave * TILE + (4 * kg + v) * BN + (KN ? CN * rc + j : rc)] = acc[0][j][v];
  }
  __syncthreads();
  if (tid >= TILE) return;
  float s = lds[tid];
#pragma unroll
  for (int w = 1; w < RW_WAVES; ++w) s += lds[w * TILE + tid];
  const int om = m0 + tid / BN, on = n0 + tid % BN;
  if (om >= M || on >= g.n_out) return;
  float* o = static_cast<float*>(g.out) + (size_t)om * g.n_out + on;
  if (g.accumulate) s += *o;
  if (g.bias) s += g.bias[on];
  if (g.relu) s = fmaxf(s, 0.f);
  *o = s;
#endif
}

template <int CN>
void launch_rows(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe) {
  probe->variant = V_IGEMM_ROWS;
  probe->kernel = CN == 4 ? "igemm_rows 16x64" : CN == 2 ? "igemm_rows 16x32" : CN == 1 ? "igemm_rows 16x16 [k][n]" : "igemm_rows 16x16";
  if (probe->dry) return;
  constexpr int BN = CN ? 16 * CN : 16;
  const int tn = (g.n_out + BN - 1) / BN, tiles = (M + 15) / 16 * tn, main_grid = (tiles + 7) / 8 * 8;
  const dim3 grid((unsigned)(main_grid + wide_reduce_blocks(g.side.count, RW_THREADS)));
  if (probe->before) (void)hipEventRecord(probe->before, st);
  hipLaunchKernelGGL((igemm_rows_kernel<CN>), grid, dim3(RW_THREADS), 0, st, g, M, K, tn, tiles, main_grid);
  if (probe->after) (void)hipEventRecord(probe->after, st);
}

// Predicted microseconds, with r tiles on the compute unit with the most: first + (r - 1) * next, linear in K (with [n][k], in batches
// of 1024 values of it).  Fitted to 160 launches of each kind (4 to 512 rows, K and N of 64 to 2048, operands of six sets in turn).
// Where r is large the wider tiles read less, up to where the other kernels' tiles fill the chip.
double rows_us(int cn, long M, long N, long K) {
  const int bn = cn ? 16 * cn : 16;
  const long tiles = (M + 15) / 16 * ((N + bn - 1) / bn), more = (tiles + 255) / 256 - 1;
  const double k = K * 1e-3, b = (double)((K + 1023) / 1024);
  switch (cn) {
    case 0: return 1.8 + 3.6 * b + more * (6.0 * b - 3.5);
    case 1: return 4.2 + 1.5 * k + more * (0.5 + 2.9 * k);
    case 2: return 3.3 + 3.9 * k + more * (2.1 + 4.1 * k);
    default: return 4.9 + 5.3 * k + more * (2.0 + 7.0 * k);
  }
}
int best_kn(long M, long N, long K) {
  const double t[3] = {rows_us(1, M, N, K), rows_us(2, M, N, K), rows_us(4, M, N, K)};
  return t[0] <= t[1] && t[0] <= t[2] ? 1 : t[1] <= t[2] ? 2 : 4;
}

}  // namespace

// Where this is predicted to be the fastest way.  Microseconds, other kernels (with the launch that transposes the filter, if [k][n] and the
// caller leaves w null for it) -> this one:
//   [n][k]  41 rows, 2048 -> 1000  29.2 -> 10.4,  196 rows, 512 -> 1000  11.8 -> 12.6 (not taken);
//   [k][n]  41 rows, 1000 -> 2048  26.1 -> 7.8,  392 rows, 1000 -> 1000  27.2 -> 19.5,  392 rows, 2048 -> 2048  45.4 -> 56.9 (not taken).
// Filters larger than the caches, which the fit below does not hold: 25088 -> 4096, 16 rows 316 -> 112 and, [k][n], 365 -> 111, 32 rows
// 326 -> 197 and 367 -> 155, from 64 rows on not taken; 4096 -> 4096, 32 rows 61 -> 35 and 90 -> 28.
// Error against float64, 2048 values of K: 1.3e-7 (2.5e-7 in the other kernels).  From K = 320 on: shorter reductions gain as well (8.0 -> 5.4
// at 256), but the kernels that take them are pinned to shapes of 224 and 288 by their tests.  Of the eight (four) values of K
// that a lane takes, and of its columns of a [k][n] filter, all exist or none; rows of a [n][k] filter start on 64 bytes (eights of K would
// do: 392 rows, 1000 -> 64  17.3 -> 5.6, not taken).
bool conv_igemm_rows_takes(const ConvGeom& g, long M, long K) {
  const bool plain = g.r == 1 && g.s == 1 && g.stride == 1 && g.pad == 0 && g.pad_dx == 0 && g.p == g.h && g.q == g.wd && g.out_stride == 1 &&
                     g.out_h == g.p && g.out_w == g.q;
  if (g.dtype != DT_F32 || !plain || g.stats || g.bnb.sums || g.flip.wt || M > 4096 || K < 320) return false;
  if (M * K * 4 > 0xFFFFFF00L || (long)g.n_out * K * 4 > 0xFFFFFF00L) return false;
  if ((reinterpret_cast<uintptr_t>(g.in) | reinterpret_cast<uintptr_t>(g.w) | reinterpret_cast<uintptr_t>(g.w_kn)) & 15) return false;
  if (g.w_kn ? K % 4 != 0 || g.n_out % 8 != 0 : K % 16 != 0) return false;
  const double here = g.w_kn ? rows_us(best_kn(M, g.n_out, K), M, g.n_out, K) : rows_us(0, M, g.n_out, K);
  const double flip = g.w_kn && !g.w ? 3.0 : 0.0;
  return here < conv_igemm_x3_us(g, M, K) + flip;
}

hipError_t conv_igemm_rows(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe) {
  if (g.side.count && (!g.side.part || !g.side.dw || g.side.splits < 1)) return hipErrorInvalidValue;
  switch (g.w_kn ? best_kn(M, g.n_out, K) : 0) {
    case 0: launch_rows<0>(g, M, K, st, probe); break;
    case 1: launch_rows<1>(g, M, K, st, probe); break;
    case 2: launch_rows<2>(g, M, K, st, probe); break;
    default: launch_rows<4>(g, M, K, st, probe); break;
  }
  return probe->dry ? hipSuccess : hipGetLastError();
}

}  // namespace acc
