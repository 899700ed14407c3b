// Implicit-GEMM convolution for fp32 storage on the bf16 matrix cores (see split3.h for the
// arithmetic), forward pass and data gradient of every layer with whole 16-channel chunks.
//
//   out[m][n] (+)= sum_k A[m][k] * W[n][k],   m = (img,p,q), k = (r,t,c), c fastest
//
// A workgroup of 4 waves (2 x 2) owns a 64*MB x 64*NB tile, each wave MB x NB blocks of 32 x 32.  The
// operands travel global memory -> registers -> LDS: on the way every fp32 value is split into its three
// bf16 parts, once per workgroup, and LDS holds three planes per operand, [row][KC bf16], from which a
// fragment is one ds_read_b128 per lane.  Two LDS stages, two register sets: the loads of chunk kc+2 are
// issued when chunk kc starts, chunk kc+1 is split and stored while chunk kc is multiplied.
//
// Bound: the matrix cores sustain 2.0-2.08 PFLOP/s in bf16 (their clock falls under load), a sixth of that, 333
// TFLOP/s, in these products; the rest is LDS traffic, splitting (13 vector instructions per two values) and the
// fixed cost of a tile.  Measured against the fp32-instruction kernel this replaces (154 TFLOP/s ceiling), forward,
// minibatch 41: 256->256 3x3 at 14x14 75.2 -> 50.2 us, 128->128 3x3 at 28x28 74.7 -> 51.0, 512->512 3x3 at 7x7
// 77.4 -> 65.6, 256->1024 1x1 at 14x14 38.6 -> 29.0, 1024->256 35.6 -> 30.0;
// error against float64 5.9e-7 -> 3.5e-7 on the first of them, smaller on all.
#include <cmath>

#include "kernels.h"
#include "dtype.h"
#include "igemm_side.h"
#include "side_wide.h"
#include "split3.h"

namespace acc {
namespace {

struct RowPos {  // decoded GEMM row
  int pix;       // img * h * wd (pixel index of the image origin)
  int iy0, ix0;  // p*stride - pad, q*stride - pad
  int ok;
};

__device__ __forceinline__ RowPos decode_row(const ConvGeom& g, int m, int M) {
  RowPos rp;
  rp.ok = m < M;
  const int mm = rp.ok ? m : 0;
  const int pq = g.p * g.q;
  const int img = mm / pq;
  const int rem = mm - img * pq;
  const int p = rem / g.q;
  const int q = rem - p * g.q;
  rp.pix = img * g.h * g.wd;
  rp.iy0 = p * g.stride - g.pad;
  rp.ix0 = q * g.stride - g.pad - g.pad_dx;
  return rp;
}

__device__ __forceinline__ size_t out_row_offset(const ConvGeom& g, int m) {
  const int pq = g.p * g.q;
  const int img = m / pq;
  const int rem = m - img * pq;
  const int p = rem / g.q;
  const int q = rem - p * g.q;
  return ((size_t)(img * g.out_h + g.out_y0 + p * g.out_stride) * g.out_w + g.out_x0 + q * g.out_stride) * g.n_out;
}

// One 32 x 32 block (rows from mr, columns from nr on) with the fp32 matrix instruction, operands straight from
// memory: for blocks whose split products are not finite, where an infinity times the zero part of a value would
// have made a NaN, or a finite value rounded to an infinite part.
__device__ __forceinline__ x3_v16f plain_block(const ConvGeom& g, int mr, int nr, int M, int K, int lane) {
  x3_v16f acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const RowPos rp = decode_row(g, mr + (lane & 31), M);
  const int n = nr + (lane & 31), k0 = (lane >> 5) * 4;
  const bool col = n < g.n_out;
  const float* w = static_cast<const float*>(g.w) + (size_t)(col ? n : 0) * K + k0;
#pragma unroll 1
  for (int kr = 0; kr < g.r; ++kr)
#pragma unroll 1
    for (int kt = 0; kt < g.s; ++kt) {
      const int iy = rp.iy0 + kr, ix = rp.ix0 + kt;
      const bool ok = rp.ok && (unsigned)iy < (unsigned)g.h && (unsigned)ix < (unsigned)g.wd;
      const float* x = static_cast<const float*>(g.in) + (size_t)(ok ? rp.pix + iy * g.wd + ix : 0) * g.c + k0;
#pragma unroll 1
      for (int c = 0; c < g.c; c += 8) {
        const bool k_ok = c + k0 < g.c;
        [[maybe_unused]] x3_v4f a = *reinterpret_cast<const x3_v4f*>(x + (k_ok ? c : 0)), b = *reinterpret_cast<const x3_v4f*>(w + (k_ok ? c : 0));
        if (!k_ok) a = b = x3_v4f{0.f, 0.f, 0.f, 0.f};
        if (!ok) a = x3_v4f{0.f, 0.f, 0.f, 0.f};
        if (!col) b = x3_v4f{0.f, 0.f, 0.f, 0.f};
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], b[u], acc, 0, 0, 0);
#endif
      }
      w += g.c;
    }
  return acc;
}

// Swizzled byte offset of 16-byte column `col` (0 or 1) of row `row` inside one plane: rows are 32 bytes (16 bf16),
// and sixteen consecutive rows read at one column lie on different ones of the 64 banks.
[[maybe_unused]] __device__ __forceinline__ int plane_at(int row, int col) { return row * 32 + ((col ^ ((row >> 3) & 1)) << 4); }

// What follows the products: a wave's MB x NB blocks, rows from mw and columns from nw on, are summed for a
// batch norm, masked, added to, biased and stored as the launch asks.
template <int MB, int NB, bool ACT>
__device__ __forceinline__ void x3_finish(const ConvGeom& g, int M, int K, int mw, int nw, int lane, x3_v16f (&acc)[MB][NB]) {
  const int half = lane >> 5;
  if (x3_any_nonfinite<MB, NB>(acc)) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) acc[i][jj] = plain_block(g, mw + 32 * i, nw + 32 * jj, M, K, lane);
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) acc[i][jj] *= kX3Unscale;
  }

  // epilogue: accumulator register v of a lane holds row 8*(v/4) + 4*(lane/32) + v%4,
  // column lane%32 of its 32x32 block
  const bool dense = g.out_stride == 1 && g.out_h == g.p && g.out_w == g.q;
  const int rows_end = (M + 63) & ~63;                   // results and sums: the blocks of sums come in pairs
  // What a block needs from memory (the old values, or the batch norm's y and x) is requested a block ahead, every
  // load unconditional (rows that do not exist read the lane's first one): one trip to memory per block, hidden
  // behind the block before, instead of one per row.  1x1 512->2048 data gradient at 7x7, minibatch 32, with the
  // batch norm's work 56.1 -> 51.9 us.
  const bool want_old = !ACT && dense && g.accumulate, want_bnb = !ACT && g.bnb.sums != nullptr;
  float pre0[2][16], pre1[2][16];
  auto block_at = [&](int b, int& n, int& mb, int& left, size_t& at0) {
    const int i = b % MB, jj = b / MB;
    n = nw + 32 * jj + (lane & 31);
    const int mr = mw + 32 * i;                          // first row of the block
    mb = mr + 4 * half;
    // the lane's first row; its other rows lie dr = 8*(v/4) + v%4 rows further on, a distance
    // that is the same for every lane
    left = n >= g.n_out ? 0 : mr + 32 <= M ? 32 : M - mb;          // rows of the lane that exist, counted from mb
    at0 = (size_t)(mb < M ? mb : 0) * g.n_out + (n < g.n_out ? n : 0);
  };
  auto request = [&](int b) {
    int n, mb, left;
    size_t at0;
    block_at(b, n, mb, left, at0);
    const float* s0 = want_old ? static_cast<const float*>(g.out) : static_cast<const float*>(g.bnb.y);
    const float* s1 = static_cast<const float*>(g.bnb.x);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int dr = 8 * (v >> 2) + (v & 3);
      const size_t at = at0 + (dr < left ? (size_t)dr * g.n_out : 0);
      pre0[b & 1][v] = s0[at];
      if (want_bnb) pre1[b & 1][v] = s1[at];
    }
  };
  if (want_old || want_bnb) request(0);
#pragma unroll
  for (int b = 0; b < MB * NB; ++b) {
    if ((want_old || want_bnb) && b + 1 < MB * NB) request(b + 1);
    int n, mb, left;
    size_t at0;
    block_at(b, n, mb, left, at0);
    const int mr = mb - 4 * half;
    if (mr >= rows_end) continue;                        // (uniform)
    const bool col = n < g.n_out;
    x3_v16f& c = acc[b % MB][b / MB];
    const size_t slab = (size_t)(mr >> 5);               // 32-row block of the whole result
    if (!ACT && g.stats) {
      // sums of the column and of its squares over the 32 rows (rows beyond M are exact zeros),
      // for the batch norm that follows.  Fixed order: the lane's 16 values, then the partner lane.
      float sum = 0.f, sq = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sum += c[v];
        sq = fmaf(c[v], c[v], sq);
      }
      sum += __shfl_xor(sum, 32);
      sq += __shfl_xor(sq, 32);
      if (lane < 32 && col) {
        g.stats[slab * g.n_out + n] = sum;
        g.stats[((size_t)g.stats_stride + slab) * g.n_out + n] = sq;
      }
    }
    if (want_bnb) {
      // Data gradient whose result is the gradient of a batch norm's ReLU output: mask it with
      // [y > 0] and leave the sums of g and g * xhat over the 32 rows for that batch norm's backward pass.
      const float mu = col ? g.bnb.mean[n] : 0.f, is = col ? g.bnb.istd[n] : 0.f;
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int dr = 8 * (v >> 2) + (v & 3);
        const bool ok = dr < left;
        const float gv = ok && pre0[b & 1][v] > 0.f ? c[v] : 0.f;
        const float xh = ok ? (pre1[b & 1][v] - mu) * is : 0.f;
        c[v] = gv;
        s0 += gv;
        s1 = fmaf(gv, xh, s1);
      }
      s0 += __shfl_xor(s0, 32);
      s1 += __shfl_xor(s1, 32);
      if (lane < 32 && col) {
        g.bnb.sums[slab * g.n_out + n] = s0;
        g.bnb.sums[((size_t)g.bnb.stride + slab) * g.n_out + n] = s1;
      }
    }
    if constexpr (ACT) {
      const float bias_n = col && g.bias ? g.bias[n] : 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        c[v] += bias_n;
        if (g.relu) c[v] = fmaxf(c[v], 0.f);
      }
    }
    if (dense) {
      if (want_old) {
#pragma unroll
        for (int v = 0; v < 16; ++v) c[v] += pre0[b & 1][v];
      }
      float* o0 = static_cast<float*>(g.out) + at0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int dr = 8 * (v >> 2) + (v & 3);
        if (dr < left) o0[(size_t)dr * g.n_out] = c[v];
      }
      continue;
    }
    // A strided result: the pixel of the lane's first row by division, the others by counting on, one carry at most per
    // step of 1 or 5 rows (sixteen divisions per block: 57 us for the data gradient of 128 channels of 55x55
    // from stride 2, 19 images; 48 so).  Old values are requested together.
    float* const first = static_cast<float*>(g.out) + out_row_offset(g, mb) + n;
    const ptrdiff_t dx = (ptrdiff_t)g.out_stride * g.n_out, dy = ((ptrdiff_t)g.out_stride * g.out_w - (ptrdiff_t)g.q * g.out_stride) * g.n_out;
    const ptrdiff_t di = ((ptrdiff_t)g.out_h * g.out_w - (ptrdiff_t)g.p * g.out_stride * g.out_w) * g.n_out;
    const bool count_on = g.q >= 5;                      // (uniform)
    const int row0 = mb / g.q, q0 = mb - row0 * g.q, p0 = row0 % g.p;
    auto rows = [&](auto&& use) {
      float* o = first;
      int q = q0, p = p0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int dr = 8 * (v >> 2) + (v & 3);
        if (v > 0) {
          if (count_on) {
            const int d = (v & 3) ? 1 : 5;
            q += d;
            o += d * dx;
            if (q >= g.q) {
              q -= g.q;
              o += dy;
              if (++p == g.p) { p = 0; o += di; }
            }
          } else {
            o = static_cast<float*>(g.out) + out_row_offset(g, mb + dr) + n;
          }
        }
        if (dr < left) use(o, v);
      }
    };
    if (!ACT && g.accumulate) {
      float old[16];
      rows([&](const float* o, int v) { old[v] = *o; });
      rows([&](float* o, int v) { *o = c[v] + old[v]; });
    } else {
      rows([&](float* o, int v) { *o = c[v]; });
    }
  }
}

// One tile of 64*MB x 64*NB, its operands staged in `lds`.
template <int MB, int NB> struct Short {
  static constexpr int BM = 64 * MB, BN = 64 * NB, KC = 16;
  static constexpr int ROWB = KC * 2;                    // bytes per row and plane
  static constexpr int A_PLANE = BM * ROWB, B_PLANE = BN * ROWB;
  static constexpr int STAGE = 3 * (A_PLANE + B_PLANE);
  static_assert(2 * STAGE >= 32 * 33 * 4, "side jobs");
};

template <int MB, int NB, bool ACT>
__device__ __forceinline__ void short_tile(const ConvGeom& g, int M, int K, int m0, int n0, char* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  using S = Short<MB, NB>;
  constexpr int BM = S::BM, BN = S::BN, KC = S::KC, ROWB = S::ROWB, A_PLANE = S::A_PLANE, B_PLANE = S::B_PLANE, STAGE = S::STAGE;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave >> 1) * 32 * MB, wn0 = (wave & 1) * 32 * NB;

  x3_v16f acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int n_chunks = (K + KC - 1) / KC;                // whole chunks but for 1x1 filters (launcher)
  constexpr int TPR = KC / 4;                            // threads per row (16 bytes of fp32 each)
  constexpr int RPP = 256 / TPR;                         // rows per pass
  constexpr int AI = BM / RPP, BI = BN / RPP;
  const int lrow = tid / TPR, lk4 = tid & (TPR - 1);
  const int margin = g.pad * g.wd + g.pad + g.pad_dx;    // pixels; the descriptor starts that far before the tensor
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;              // beyond any descriptor range: reads as zero
  uint32_t a_voff[AI], a_mask[AI], b_voff[BI];
  // 1x1, stride 1, no padding: GEMM row m is pixel m, nothing to decode
  const bool plain = g.r == 1 && g.s == 1 && g.stride == 1 && g.pad == 0 && g.pad_dx == 0 && g.p == g.h && g.q == g.wd;
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int m = m0 + lrow + RPP * i;
    if (plain) {
      a_voff[i] = (uint32_t)(m < M ? m : 0) * (uint32_t)(g.c * 4) + lk4 * 16;
      a_mask[i] = m < M ? 1u : 0u;
      continue;
    }
    const RowPos rp = decode_row(g, m, M);
    a_voff[i] = (uint32_t)(rp.pix + rp.iy0 * g.wd + rp.ix0 + margin) * (uint32_t)(g.c * 4) + lk4 * 16;
    uint32_t mask = 0;
    for (int kr = 0; kr < g.r; ++kr)
      for (int kt = 0; kt < g.s; ++kt) {
        const bool ok = rp.ok && (unsigned)(rp.iy0 + kr) < (unsigned)g.h && (unsigned)(rp.ix0 + kt) < (unsigned)g.wd;
        mask |= (ok ? 1u : 0u) << (kr * g.s + kt);
      }
    a_mask[i] = mask;
  }
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int n = n0 + lrow + RPP * i;
    b_voff[i] = n < g.n_out ? (uint32_t)n * (uint32_t)(K * 4) + lk4 * 16 : OUTSIDE;
  }
  const size_t margin_bytes = (size_t)margin * g.c * 4;
  const size_t a_bytes = margin_bytes + (size_t)g.n_img * g.h * g.wd * g.c * 4;
  __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(g.in)) - margin_bytes, 0, (int)(uint32_t)a_bytes, 0x00020000);
  __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(g.w), 0, (int)(uint32_t)((size_t)g.n_out * K * 4), 0x00020000);

  struct Regs { x3_v4u a[AI], b[BI]; } R0, R1;
  int kr = 0, kt = 0, c0 = 0, kb = 0;     // tap, channel offset and filter offset of the chunk whose loads are issued next (uniform)
  auto advance = [&]() {
    kb += KC * 4;
    c0 += KC;
    if (c0 == g.c) {
      c0 = 0;
      if (++kt == g.s) { kt = 0; ++kr; }
    }
  };
  auto load = [&](Regs& R) {
    const int tap = kr * g.s + kt;
    const int soff_a = ((kr * g.wd + kt) * g.c + c0) * 4;
    const bool k_ok = c0 + lk4 * 4 < g.c;                // (1x1 filters: K need not be whole chunks)
#pragma unroll
    for (int i = 0; i < AI; ++i)
      R.a[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_a, ((((a_mask[i] >> tap) & 1u) != 0) & k_ok) ? a_voff[i] : OUTSIDE, soff_a, 0);
#pragma unroll
    for (int i = 0; i < BI; ++i) R.b[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_b, b_voff[i], kb, 0);
    advance();
  };
  const int st_at = plane_at(lrow, lk4 >> 1) + (lk4 & 1) * 8;   // rows RPP further on keep the swizzle
  static_assert(RPP % 16 == 0, "swizzle period");
  auto put = [&](const x3_v4u& x, char* at, int plane) {
    uint32_t h0, m0_, l0, h1, m1_, l1;
    x3_split(__uint_as_float(x[0]), __uint_as_float(x[1]), h0, m0_, l0);
    x3_split(__uint_as_float(x[2]), __uint_as_float(x[3]), h1, m1_, l1);
    *reinterpret_cast<x3_v2u*>(at) = x3_v2u{h0, h1};
    *reinterpret_cast<x3_v2u*>(at + plane) = x3_v2u{m0_, m1_};
    *reinterpret_cast<x3_v2u*>(at + 2 * plane) = x3_v2u{l0, l1};
  };
  auto store = [&](const Regs& R, int buf) {
    char* as = lds + buf * STAGE + st_at;
#pragma unroll
    for (int i = 0; i < AI; ++i) put(R.a[i], as + i * RPP * ROWB, A_PLANE);
    char* bs = as + 3 * A_PLANE;
#pragma unroll
    for (int i = 0; i < BI; ++i) put(R.b[i], bs + i * RPP * ROWB, B_PLANE);
  };
  const int fra = wm0 + (lane & 31), frb = wn0 + (lane & 31), half = lane >> 5;
  // The largest product of a step, h*h, goes into one set of accumulators, the five small ones into another:
  // an addition to the large sum rounds once per 16 products, and the small sums' roundings are 2^8 smaller.
  x3_v16f accs[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) accs[i][j][v] = 0.f;
  // One step: the chunk in LDS stage `buf` is multiplied, the chunk in registers R is split and stored into the
  // other stage.  The h*h products of the chunk before are held back (ph_a, ph_b) until this chunk's fragments
  // have been requested; the splitting is spread over the matrix instructions.
  x3_v4u ph_a[1][MB], ph_b[1][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i) ph_a[0][i] = x3_v4u{0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < NB; ++j) ph_b[0][j] = x3_v4u{0, 0, 0, 0};
  auto held = [&]() {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) acc[i][jj] = x3_mfma(ph_a[0][i], ph_b[0][jj], acc[i][jj]);
  };
  auto step = [&](int buf, const Regs* R, Regs* L) {
    const char* as = lds + buf * STAGE + plane_at(fra, half);
    const char* bs = lds + buf * STAGE + 3 * A_PLANE + plane_at(frb, half);
    x3_v4u a[3][MB], b[3][NB];
    auto rd_a = [&](int p) {
#pragma unroll
      for (int i = 0; i < MB; ++i) a[p][i] = *reinterpret_cast<const x3_v4u*>(as + p * A_PLANE + i * 32 * ROWB);
    };
    auto rd_b = [&](int p) {
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) b[p][jj] = *reinterpret_cast<const x3_v4u*>(bs + p * B_PLANE + jj * 32 * ROWB);
    };
    __builtin_amdgcn_sched_barrier(0);
    rd_a(2); rd_b(0); rd_a(0); rd_b(2); rd_a(1); rd_b(1);
    __builtin_amdgcn_sched_barrier(0);
    held();
    if (L) load(*L);
    if (R) store(*R, buf ^ 1);
    x3_product<2, 0, MB, NB>(a, b, accs);
    x3_product<0, 2, MB, NB>(a, b, accs);
    x3_product<1, 1, MB, NB>(a, b, accs);
    x3_product<1, 0, MB, NB>(a, b, accs);
    x3_product<0, 1, MB, NB>(a, b, accs);
#pragma unroll
    for (int i = 0; i < MB; ++i) ph_a[0][i] = a[0][i];
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) ph_b[0][jj] = b[0][jj];
    if (R) {
      constexpr int V = (26 * (AI + BI) + 6 * MB * NB - 1) / (6 * MB * NB) + 1;     // vector instructions per matrix instruction
#pragma unroll
      for (int u = 0; u < 6 * MB * NB; ++u) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
        if (u == 0 && L) __builtin_amdgcn_sched_group_barrier(0x020, AI + BI, 0);
        if (u % (2 * MB * NB) == 2 * MB * NB - 1) __builtin_amdgcn_sched_group_barrier(0x200, AI + BI, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // One barrier per chunk: it says that chunk kc+1 is in LDS and that everybody is done with chunk kc,
  // whose stage chunk kc+2 may overwrite.
  load(R0);
  if (n_chunks > 1) load(R1);
  store(R0, 0);
  __syncthreads();
  int j = 0;
  for (; j + 4 <= n_chunks; j += 2) {        // steady state: every load and store unconditional
    step(0, &R1, &R0);
    __syncthreads();
    step(1, &R0, &R1);
    __syncthreads();
  }
  for (; j < n_chunks; j += 2) {
    if (j + 2 < n_chunks) load(R0);
    step(0, nullptr, nullptr);
    if (j + 1 < n_chunks) store(R1, 1);
    __syncthreads();
    if (j + 1 >= n_chunks) break;
    if (j + 3 < n_chunks) load(R1);
    step(1, nullptr, nullptr);
    if (j + 2 < n_chunks) store(R0, 0);
    __syncthreads();
  }
  held();
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) acc[i][jj] += accs[i][jj];
  x3_finish<MB, NB, ACT>(g, M, K, m0 + wm0, n0 + wn0, lane, acc);
#else
  (void)&decode_row; (void)&out_row_offset; (void)&plain_block;
#endif
}

template <int MB, int NB, bool ACT>
__global__ __launch_bounds__(256, 2) void igemm_x3_kernel(ConvGeom g, int M, int K, int n_tiles_n,
                                                                              int n_tiles, int main_grid) {
  using S = Short<MB, NB>;
  __shared__ __attribute__((aligned(1024))) char lds[2 * S::STAGE];
  if ((int)blockIdx.x >= main_grid) {
    igemm_side_jobs<float>(g, (int)blockIdx.x - main_grid, lds);
    return;
  }
  // Forward products and data gradients are the critical path of an iteration; a weight gradient may run
  // beside them on a stream of its own at the default wave priority.
  __builtin_amdgcn_s_setprio(3);
  // XCD-aware tile order: consecutive workgroup ids land on different XCDs, so give each XCD a
  // contiguous range of tiles (neighbouring tiles share operand rows in its L2).
  const int per_xcd = main_grid >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= n_tiles) return;
  const int tile_m = tile / n_tiles_n, tile_n = tile - tile_m * n_tiles_n;
  short_tile<MB, NB, ACT>(g, M, K, tile_m * S::BM, tile_n * S::BN, lds);
}

// The parts of a strided data gradient in one launch.  Alone, a part of a 3x3 stride-2 filter is a quarter of the rows
// and one to four taps: too few tiles and too short a K to fill the chip or to pay for a launch.  Together their tiles
// even out, the parts with the longest K first, and each XCD keeps the same range of rows of every part: the parts
// read the same rows of the gradient.  128 -> 128 3x3 stride 2 on 55x55,
// 19 images, with the sub-filters' launches: 79 us apart, 57 together, 48 with the counted rows of the epilogue above.
constexpr int kX3Parts = 4;
struct X3Parts {
  ConvGeom g[kX3Parts];
  int M[kX3Parts], K[kX3Parts], tiles[kX3Parts], per_xcd[kX3Parts];
};

template <int MB, int NB>
__global__ __launch_bounds__(256, 2) void igemm_x3_parts_kernel(X3Parts ps, int n_tiles_n, int main_grid) {
  using S = Short<MB, NB>;
  __shared__ __attribute__((aligned(1024))) char lds[2 * S::STAGE];
  if ((int)blockIdx.x >= main_grid) {
    igemm_side_jobs<float>(ps.g[0], (int)blockIdx.x - main_grid, lds);
    return;
  }
  __builtin_amdgcn_s_setprio(3);
  int i = 0, at = blockIdx.x >> 3;             // place in the XCD's list: its tiles of part 0, of part 1, ...
  for (; i < kX3Parts - 1 && at >= ps.per_xcd[i]; ++i) at -= ps.per_xcd[i];
  const int tile = (blockIdx.x & 7) * ps.per_xcd[i] + at;
  if (tile >= ps.tiles[i]) return;
  const int tile_m = tile / n_tiles_n, tile_n = tile - tile_m * n_tiles_n;
  short_tile<MB, NB, false>(ps.g[i], ps.M[i], ps.K[i], tile_m * S::BM, tile_n * S::BN, lds);
}

// ---- long reductions: eight waves, each 64 x 64 (2 x 2 blocks), the steps of K dealt out to groups of waves
//
// What a step costs besides its 24 matrix instructions per wave is LDS traffic (12 KB read per wave, 96 bytes
// per operand row written) and the splitting of the operand rows, so a wave's tile is as large as its
// registers allow, and a tile of 64*WM x 64*WN is shared by KS = 8 / (WM*WN) groups that take every KS-th
// step: the chip is filled by tiles x KS even where the minibatch gives few tiles.  Fragments are fetched one
// step ahead: while step j is multiplied out of registers, step j+1 is read from LDS, step j+2 is split and
// stored, later loads are issued.  Nothing in a step waits for anything else of that step.  At the end the groups exchange their sums through LDS, each adding
// up and writing some of the blocks.
//
// WINDOW: stride-1 convolutions with r x r > 1 taps whose output has the size of the input.  GEMM row m is
// pixel m there, and tap (kr, kt) reads pixel m + (kr - pad) * wd + (kt - pad): for the rows of a tile all taps
// read one window of consecutive pixels.  The window's 16 channels of a step are fetched, split and stored
// once, by the whole workgroup, and serve all r*r taps and all groups; a lane whose tap falls into the padding
// is pointed at a row of zeros.
template <int WM, int WN, bool WINDOW>
struct Deep {
  static constexpr int KS = 8 / (WM * WN), GT = 64 * WM * WN;        // groups, threads of a group
  static constexpr int BM = 64 * WM, BN = 64 * WN;
  static constexpr int WROWS = 256, WPLANE = (WROWS + 1) * 32, WBUF = WINDOW ? 3 * WPLANE : 0;   // largest window, a row of zeros
  static constexpr int AP = WINDOW ? 0 : BM * 32, BP = BN * 32, STAGE = 3 * (AP + BP);
  static constexpr int NST = GT == 64 ? 1 : 2;                       // a group of one wave needs no second stage: its LDS accesses keep their order
  static constexpr int MAIN = 2 * WBUF + KS * NST * STAGE;
  static constexpr int NQ = KS < 4 ? KS : 4, BPQ = 4 / NQ;           // groups that finish blocks, blocks each
  static constexpr int RED = NQ * (KS - 1) * WM * WN * BPQ * 16 * 64 * 4;
  static constexpr int LDS = MAIN > RED ? MAIN : RED;
};

template <int WM, int WN, bool WINDOW, bool ACT>
__global__ __launch_bounds__(512, 1) void igemm_x3_deep_kernel(ConvGeom g, int M, int K, int n_tiles_n, int n_tiles, int main_grid) {
  using D = Deep<WM, WN, WINDOW>;
  [[maybe_unused]] constexpr int KS = D::KS, GT = D::GT;
  __shared__ __attribute__((aligned(1024))) char lds[D::LDS];
  if ((int)blockIdx.x >= main_grid) {
    static_assert(D::LDS >= wide_scratch<float>(512), "side jobs");
    wide_side_jobs<float, 512>(g.side, g.flip, (int)blockIdx.x - main_grid, lds);
    return;
  }
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_s_setprio(3);
  const int per_xcd = main_grid >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= n_tiles) return;
  const int tile_m = tile / n_tiles_n, tile_n = tile - tile_m * n_tiles_n;
  const int m0 = tile_m * D::BM, n0 = tile_n * D::BN;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
  const int grp = __builtin_amdgcn_readfirstlane(tid / GT), gt = tid & (GT - 1);
  const int gw = __builtin_amdgcn_readfirstlane((tid >> 6) & (WM * WN - 1));   // wave of the group
  const int wm0 = (gw / WN) * 64, wn0 = (gw % WN) * 64;
  const int taps = g.r * g.s, n_steps = (K + 15) >> 4;
  constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;              // beyond any descriptor range: reads as zero
  const int margin = WINDOW ? 0 : g.pad * g.wd + g.pad + g.pad_dx;   // pixels; the descriptor starts that far before the tensor
  const size_t margin_bytes = (size_t)margin * g.c * 4;
  __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(reinterpret_cast<const char*>(g.in)) - margin_bytes, 0,
      (int)(uint32_t)(margin_bytes + (size_t)g.n_img * g.h * g.wd * g.c * 4), 0x00020000);
  __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(g.w), 0, (int)(uint32_t)((size_t)g.n_out * K * 4), 0x00020000);
  auto tap_mask = [&](const RowPos& rp) {
    uint32_t mk = 0;
    for (int kr = 0; kr < g.r; ++kr)
      for (int kt = 0; kt < g.s; ++kt) {
        const bool ok = rp.ok && (unsigned)(rp.iy0 + kr) < (unsigned)g.h && (unsigned)(rp.ix0 + kt) < (unsigned)g.wd;
        mk |= (ok ? 1u : 0u) << (kr * g.s + kt);
      }
    return mk;
  };

  // ---- loads: 16 bytes (four values of K) per thread and row
  constexpr int RPP = GT / 4, AI = WINDOW ? 0 : D::BM / RPP, BI = D::BN / RPP;   // rows per pass of the group; passes
  constexpr int AN = AI > 0 ? AI : 1;
  uint32_t a_voff[AN], a_mask[AN], b_voff[BI];
  const bool plain = g.r == 1 && g.s == 1 && g.stride == 1 && g.pad == 0 && g.pad_dx == 0 && g.p == g.h && g.q == g.wd;
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int m = m0 + (gt >> 2) + RPP * i;
    if (plain) {      // 1x1, stride 1, no padding: GEMM row m is pixel m
      a_voff[i] = (uint32_t)(m < M ? m : 0) * (uint32_t)(g.c * 4) + (gt & 3) * 16;
      a_mask[i] = m < M ? 1u : 0u;
      continue;
    }
    const RowPos rp = decode_row(g, m, M);
    a_voff[i] = (uint32_t)(rp.pix + rp.iy0 * g.wd + rp.ix0 + margin) * (uint32_t)(g.c * 4) + (gt & 3) * 16;
    a_mask[i] = tap_mask(rp);
  }
#pragma unroll
  for (int i = 0; i < BI; ++i) {
    const int n = n0 + (gt >> 2) + RPP * i;
    b_voff[i] = n < g.n_out ? (uint32_t)n * (uint32_t)(K * 4) + (gt & 3) * 16 : OUTSIDE;
  }
  // One register set where a thread loads eight vectors per step, else two.
  constexpr int NR = AI + BI > 6 ? 1 : 2;
  struct Regs { x3_v4u a[AN], b[BI]; } R0, R1_;
  Regs& R1 = NR == 2 ? R1_ : R0;
  // The group's steps.  WINDOW: every KS-th of the sequence in which the taps run fastest.  Else: a range of the
  // sequence in which the channels run fastest (the next tap of a filter row continues where the channels of the
  // one before end, so offsets only jump from one filter row to the next).
  const int first = WINDOW ? grp : (int)((long)n_steps * grp / KS);
  const int mine = WINDOW ? (n_steps - grp + KS - 1) / KS : (int)((long)n_steps * (grp + 1) / KS) - first;
  const int rounds = (n_steps + KS - 1) / KS;            // the most steps of any group
  int lw, ltap, lkt, lc, soff_a = 0, soff_b = 0;
  if constexpr (WINDOW) {
    lw = first / taps; ltap = first - lw * taps;
    lkt = lc = 0;
  } else {
    const int spt = (g.c + 15) >> 4;
    ltap = first / spt; lc = (first - ltap * spt) * 16;
    lkt = ltap % g.s; lw = 0;
    soff_a = (((ltap / g.s) * g.wd + lkt) * g.c + lc) * 4;
    soff_b = first * 64;
  }
  const int row_jump = (g.wd - g.s) * g.c * 4;
  int cw = lw, ctap = ltap, ckr = ctap / g.s, ckt = ctap - (ctap / g.s) * g.s;   // WINDOW: the step that is read from LDS next
  auto load = [&](Regs& R) {
    if constexpr (WINDOW) {
      const int so = (ltap * g.c + lw * 16) * 4;
#pragma unroll
      for (int i = 0; i < BI; ++i) R.b[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_b, b_voff[i], so, 0);
      ltap += KS;                  // KS <= taps
      const bool wrap = ltap >= taps;
      ltap -= wrap ? taps : 0;
      lw += wrap ? 1 : 0;
    } else {
      const bool k_ok = lc + (gt & 3) * 4 < g.c;         // (1x1 filters: K need not be whole steps)
#pragma unroll
      for (int i = 0; i < AI; ++i)
        R.a[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_a, ((((a_mask[i] >> ltap) & 1u) != 0) & k_ok) ? a_voff[i] : OUTSIDE, soff_a, 0);
#pragma unroll
      for (int i = 0; i < BI; ++i) R.b[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_b, b_voff[i], soff_b, 0);
      soff_b += 64;
      lc += 16;
      const bool wrap = lc == g.c;
      lc = wrap ? 0 : lc;
      ltap += wrap ? 1 : 0;
      lkt += wrap ? 1 : 0;
      const bool down = lkt == g.s;
      lkt = down ? 0 : lkt;
      soff_a += 64 + (down ? row_jump : 0);
    }
  };
  // ---- split and store
  auto put = [&](const x3_v4u& x, char* at, int plane) {
    uint32_t h0, m0_, l0, h1, m1_, l1;
    x3_split(__uint_as_float(x[0]), __uint_as_float(x[1]), h0, m0_, l0);
    x3_split(__uint_as_float(x[2]), __uint_as_float(x[3]), h1, m1_, l1);
    *reinterpret_cast<x3_v2u*>(at) = x3_v2u{h0, h1};
    *reinterpret_cast<x3_v2u*>(at + plane) = x3_v2u{m0_, m1_};
    *reinterpret_cast<x3_v2u*>(at + 2 * plane) = x3_v2u{l0, l1};
  };
  char* const lds_g = lds + 2 * D::WBUF + grp * (D::NST * D::STAGE);
  static_assert(RPP % 16 == 0, "swizzle period");
  const int st_at = plane_at(gt >> 2, (gt & 3) >> 1) + (gt & 1) * 8;
  auto store = [&](const Regs& R, int buf) {
    char* as = lds_g + (buf & (D::NST - 1)) * D::STAGE + st_at;
#pragma unroll
    for (int i = 0; i < AI; ++i) put(R.a[i], as + i * RPP * 32, D::AP);
    char* bs = as + 3 * D::AP;
#pragma unroll
    for (int i = 0; i < BI; ++i) put(R.b[i], bs + i * RPP * 32, D::BP);
  };
  // ---- the window: thread -> 16 bytes of rows tid/4 and tid/4 + 128
  x3_v4u W[2];
  uint32_t w_voff[2], mask[2];
  const int w_at = plane_at(tid >> 2, (tid & 3) >> 1) + (tid & 1) * 8;
  if constexpr (WINDOW) {
    const int reach = g.pad * g.wd + g.pad;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = (tid >> 2) + 128 * i, px = m0 - reach + row;
      w_voff[i] = row < D::BM + 2 * reach && px >= 0 && px < M ? (uint32_t)px * (uint32_t)(g.c * 4) + (tid & 3) * 16 : OUTSIDE;
      mask[i] = tap_mask(decode_row(g, m0 + wm0 + 32 * i + (lane & 31), M));
    }
    if (tid < 12)      // the rows of zeros, one per stage and plane
      *reinterpret_cast<x3_v4u*>(lds + (tid / 6) * D::WBUF + ((tid % 6) >> 1) * D::WPLANE + D::WROWS * 32 + (tid & 1) * 16) = x3_v4u{0, 0, 0, 0};
  }
  auto load_window = [&](int w) {
#pragma unroll
    for (int i = 0; i < 2; ++i) W[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_a, w_voff[i], w * 64, 0);
  };
  auto store_window = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) put(W[i], lds + buf * D::WBUF + w_at + i * (128 * 32), D::WPLANE);
  };
  // ---- fragments and products
  struct Frags { x3_v4u a[3][2], b[3][2]; } F0, F1;
  const int fa_at = plane_at(wm0 + (lane & 31), half), fb_at = plane_at(wn0 + (lane & 31), half);
  int at[2] = {fa_at, fa_at + 32 * 32};
  const int ks_r = KS / g.s, ks_t = KS - ks_r * g.s;
  auto aim = [&]() {               // WINDOW: where the rows of the step lie that is read next
    if constexpr (WINDOW) {
      const int shift = ckr * g.wd + ckt, wb = (cw & 1) * D::WBUF;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        at[i] = wb + plane_at((mask[i] >> ctap) & 1u ? wm0 + (lane & 31) + 32 * i + shift : D::WROWS, half);
        asm volatile("" : "+v"(at[i]));      // worked out here, not where it is used
      }
      // KS taps on, without branches: all ones where there is no wrap
      ckt += ks_t - g.s;
      ckr += ks_r + 1;
      const int same_row = ckt >> 31;
      ckt += g.s & same_row;
      ckr += same_row;
      ctap += KS - taps;
      const int same_window = ctap >> 31;
      ctap += taps & same_window;
      cw += 1 + same_window;
      ckr -= g.r & ~same_window;
    }
  };
  auto read = [&](Frags& F, int buf) {
    const char* st = lds_g + (buf & (D::NST - 1)) * D::STAGE;
    const char* as = WINDOW ? lds : st;
    const char* bs = st + 3 * D::AP + fb_at;
    constexpr int APL = WINDOW ? D::WPLANE : D::AP;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        F.a[p][i] = *reinterpret_cast<const x3_v4u*>(as + p * APL + at[i]);
        F.b[p][i] = *reinterpret_cast<const x3_v4u*>(bs + p * D::BP + i * (32 * 32));
      }
  };
  x3_v16f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto multiply = [&](const Frags& F) {
    x3_product<2, 0, 2, 2>(F.a, F.b, acc);
    x3_product<0, 2, 2, 2>(F.a, F.b, acc);
    x3_product<1, 1, 2, 2>(F.a, F.b, acc);
    x3_product<1, 0, 2, 2>(F.a, F.b, acc);
    x3_product<0, 1, 2, 2>(F.a, F.b, acc);
    x3_product<0, 0, 2, 2>(F.a, F.b, acc);
  };
  auto sync = [&]() {              // a group of one wave shares nothing with the others but the window
    if constexpr (D::NST == 2 || WINDOW) __syncthreads();
  };
  // Step j: fragments F multiplied, fragments of j+1 read from stage (j+1)&1 into G, step j+2 (in R) stored into
  // stage j&1, whose last reader was step j-1's read of j; its registers are loaded with step j+2+NR.
  auto step = [&](const Frags& F, Frags& G, Regs& R, int par) {
    __builtin_amdgcn_sched_barrier(0);
    read(G, par ^ 1);
    x3_product<2, 0, 2, 2>(F.a, F.b, acc);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    aim();                         // for the next step, behind matrix instructions: nothing stands between the barrier and them
    store(R, par);
    load(R);
    x3_product<0, 2, 2, 2>(F.a, F.b, acc);
    x3_product<1, 1, 2, 2>(F.a, F.b, acc);
    x3_product<1, 0, 2, 2>(F.a, F.b, acc);
    x3_product<0, 1, 2, 2>(F.a, F.b, acc);
    x3_product<0, 0, 2, 2>(F.a, F.b, acc);
    constexpr int V = (26 * (AI + BI) + (WINDOW ? 20 : 6) + 19) / 20;
#pragma unroll
    for (int u = 0; u < 20; ++u) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
      if (u >= 8) __builtin_amdgcn_sched_group_barrier(0x200, (3 * (AI + BI) + 23) / 24, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Window w + 1 goes into the stage of window w - 1: from the round on after the last step of w - 1 has been
  // read, one round before its own first step is read (taps >= 2 * KS - 1 steps per window).  Step s is read
  // in round s / KS - 1.
  const int n_win = g.c >> 4;
  int w_next = 1, w_round = -1;
  auto window = [&](int round) {
    if constexpr (WINDOW) {
      if (round == w_round && w_next < n_win) {
        store_window(w_next & 1);
        if (w_next + 1 < n_win) load_window(w_next + 1);
        w_round = (taps * w_next - 1) / KS;
        ++w_next;
      }
    }
  };
  if constexpr (WINDOW) load_window(0);
  if (mine > 0) load(R0);
  if (NR == 2 && mine > 1) load(R1);
  if constexpr (WINDOW) {
    store_window(0);
    if (n_win > 1) load_window(1);
  }
  if (mine > 0) store(R0, 0);
  if (mine > NR) load(R0);
  sync();
  window(-1);
  aim();
  if (mine > 0) read(F0, 0);
  aim();
  if (mine > 1) store(R1, 1);
  if (mine > NR + 1) load(R1);
  sync();
  int j = 0;
  for (; j + 4 + NR <= mine; j += 2) {   // steady state: every load and store unconditional
    window(j);
    step(F0, F1, R0, 0);
    sync();
    window(j + 1);
    step(F1, F0, R1, 1);
    sync();
  }
  for (; j < rounds; j += 2) {
    window(j);
    if (j + 1 < mine) read(F1, 1);
    aim();
    if (j + 2 < mine) store(R0, 0);
    if (j + 2 + NR < mine) load(R0);
    if (j < mine) multiply(F0);
    sync();
    if (j + 1 >= rounds) break;
    window(j + 1);
    if (j + 2 < mine) read(F0, 0);
    aim();
    if (j + 3 < mine) store(R1, 1);
    if (j + 3 + NR < mine) load(R1);
    if (j + 1 < mine) multiply(F1);
    sync();
  }
  // ---- group q < NQ adds up the blocks BPQ*q ... of all wave positions, the groups' sums in their order after its own
  constexpr int BLK = 16 * 64, PER = WM * WN * D::BPQ * BLK;      // floats of a block, of one (to, from) pair of groups
  float* const red = reinterpret_cast<float*>(lds) + gw * (D::BPQ * BLK) + lane;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < D::NQ; ++q) {
    if (q == grp) continue;
    float* to = red + (q * (KS - 1) + (grp < q ? grp : grp - 1)) * PER;
#pragma unroll
    for (int b = 0; b < D::BPQ; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) to[b * BLK + v * 64] = acc[(q * D::BPQ + b) >> 1][(q * D::BPQ + b) & 1][v];
  }
  __syncthreads();
  if (KS > D::NQ && grp >= D::NQ) return;
  x3_v16f c[1][D::BPQ];            // BPQ = 2: one row block, two column blocks; BPQ = 1: one block
#pragma unroll
  for (int q = 0; q < D::NQ; ++q)
    if (q == grp) {
#pragma unroll
      for (int b = 0; b < D::BPQ; ++b) c[0][b] = acc[(q * D::BPQ + b) >> 1][(q * D::BPQ + b) & 1];
    }
#pragma unroll
  for (int u = 0; u < KS - 1; ++u)
#pragma unroll
    for (int b = 0; b < D::BPQ; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) c[0][b][v] += red[(grp * (KS - 1) + u) * PER + b * BLK + v * 64];
  const int blk = grp * D::BPQ;
  x3_finish<1, D::BPQ, ACT>(g, M, K, m0 + wm0 + 32 * (blk >> 1), n0 + wn0 + 32 * (blk & 1), lane, c);
#else
  (void)&decode_row;
#endif
}

template <int WM, int WN, bool WINDOW>
void launch_deep(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe) {
  probe->variant = WINDOW ? V_IGEMM_X3_WINDOW : V_IGEMM_X3_DEEP;
  probe->kernel = WINDOW ? "igemm_x3_deep window 128x64" : WM * WN == 4 ? "igemm_x3_deep 128x128" : WM * WN == 2 ? "igemm_x3_deep 128x64"
                                                                                                              : "igemm_x3_deep 64x64";
  if (probe->dry) return;
  const long side_blocks = wide_side_blocks(g.side, g.flip, 512);
  using D = Deep<WM, WN, WINDOW>;
  const int tm = (M + D::BM - 1) / D::BM, tn = (g.n_out + D::BN - 1) / D::BN;
  const int tiles = tm * tn, main_grid = (tiles + 7) / 8 * 8;
  const dim3 grid((unsigned)(main_grid + side_blocks));
  if (probe->before) (void)hipEventRecord(probe->before, st);
  if (g.bias || g.relu)
    hipLaunchKernelGGL((igemm_x3_deep_kernel<WM, WN, WINDOW, true>), grid, dim3(512), 0, st, g, M, K, tn, tiles, main_grid);
  else
    hipLaunchKernelGGL((igemm_x3_deep_kernel<WM, WN, WINDOW, false>), grid, dim3(512), 0, st, g, M, K, tn, tiles, main_grid);
  if (probe->after) (void)hipEventRecord(probe->after, st);
}

template <int MB, int NB>
void launch_short(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe, long side_blocks) {
  probe->variant = V_IGEMM_X3;
  probe->kernel = MB == 2 ? "igemm_x3 128x128" : "igemm_x3 64x64";
  if (probe->dry) return;
  const int tm = (M + 64 * MB - 1) / (64 * MB), tn = (g.n_out + 64 * NB - 1) / (64 * NB);
  const int tiles = tm * tn, main_grid = (tiles + 7) / 8 * 8;
  const dim3 grid((unsigned)(main_grid + side_blocks));
  if (probe->before) (void)hipEventRecord(probe->before, st);
  if (g.bias || g.relu)
    hipLaunchKernelGGL((igemm_x3_kernel<MB, NB, true>), grid, dim3(256), 0, st, g, M, K, tn, tiles, main_grid);
  else
    hipLaunchKernelGGL((igemm_x3_kernel<MB, NB, false>), grid, dim3(256), 0, st, g, M, K, tn, tiles, main_grid);
  if (probe->after) (void)hipEventRecord(probe->after, st);
}

// Which kernel: the one with the smallest predicted time, in microseconds.  With steps = steps of K (16 values; 32 in the direct
// kernel with the fp32 instruction) per group of waves, and tiles counted on the compute unit with the most,
//   one workgroup per compute unit:  base + first + first_step * steps + (tiles - 1) * (next + next_step * steps) + memory,
//   several (r <= per_cu resident):  base + (compute^2 + memory^2)^(1/2),  compute = the sum over rounds of
//                                    max(first + first_step * steps, r * (next + next_step * steps)),
// taps more per tile for filters larger than 1x1, and memory = per_mb_read * MB of both operands + per_mb_written * MB of the
// result, each once.  The constants are fitted to 500 measured launches (the layers of the ResNets at minibatches 1 to 128 and
// random ones, every kernel on each; profiles/conv_f32_kernels_by_shape.txt), six sets of tensors in turn, so that large operands
// come from memory and not from the caches, as in a program that touches other tensors between two calls: median errors of 1-4 %,
// the choice is within 0.5 % of the best on average, 12 % at most (on the same tensors again and again: 0.7 %, 19 %).  The fp32
// instruction's kernel is kept for the launches where it is still the faster one, small ones above all (256->64 1x1 at 56x56, 4
// images 7.6 against 8.9 us) and those that write much more than they compute (64->256, 32 images 46.5 against 48.7, 128 images 165
// against 176); it wins ties within 2 % and 0.3 us.  A function of the shape and the alignment only, never of the swap plan (pool offsets
// are multiples of 256).
struct Kind {
  int bm, bn, ks, kc, per_cu;
  double base, first, first_step, next, next_step, taps, per_mb_read, per_mb_written;
};
enum { X3_128 = 0, X3_64, X3_WINDOW, X3_DEEP_2x1, X3_DEEP_2x2, X3_DEEP_1x1, X3_KINDS, F32_ONE = X3_KINDS, F32_TWO, KINDS };
constexpr Kind kKinds[KINDS] = {
    {128, 128, 1, 16, 2, 3.79, 3.34, 0.744, 1.78, 0.644, 0.78, 0.139, 0.324},    // igemm_x3_kernel<2, 2>
    {64, 64, 1, 16, 5, 4.19, 0.154, 0.374, 0.093, 0.241, 0.046, 0.107, 0.335},   // igemm_x3_kernel<1, 1>
    {128, 64, 4, 16, 1, 2.49, 3.90, 0.973, 3.39, 1.166, 0.47, 0.013, 0.414},     // igemm_x3_deep_kernel<2, 1, window>
    {128, 64, 4, 16, 1, 5.47, 0.83, 1.137, 3.38, 1.683, 2.02, 0.148, 0.119},     // igemm_x3_deep_kernel<2, 1>
    {128, 128, 2, 16, 1, 5.65, 1.72, 0.843, 3.56, 1.297, 0.76, 0.076, 0.160},    // igemm_x3_deep_kernel<2, 2>
    {64, 64, 8, 16, 1, 4.19, 1.53, 1.449, 3.10, 1.861, 1.55, 0.118, 0.150},      // igemm_x3_deep_kernel<1, 1>
    {64, 64, 1, 32, 4, 2.72, 4.73, 0.017, 0.597, 0.496, 0.08, 0.134, 0.134},     // igemm_kernel<direct>, fp32
    {64, 64, 2, 32, 1, 3.19, 0.134, 0.995, 0.134, 0.995, 1.09, 0, 0.234},        // igemm_kernel<direct, two groups>: one tile at most
};
double predicted_us(const Kind& k, const ConvGeom& g, long M, long K) {
  const long N = g.n_out;
  const long tiles = ((M + k.bm - 1) / k.bm) * ((N + k.bn - 1) / k.bn), steps = ((K + k.kc - 1) / k.kc + k.ks - 1) / k.ks;
  const long most = (tiles + 255) / 256;                 // tiles of the busiest compute unit
  const double first = k.first + k.first_step * steps, next = k.next + k.next_step * steps, more = g.r * g.s > 1 ? k.taps * most : 0;
  const double read = 4e-6 * ((double)g.n_img * g.h * g.wd * g.c + (double)N * K), written = 4e-6 * (double)M * N;
  const double memory = k.per_mb_read * read + k.per_mb_written * written;
  if (k.per_cu == 1) return k.base + first + (most - 1) * next + more + memory;
  auto round = [&](long r) { return r == 0 ? 0.0 : first > r * next ? first : r * next; };
  const double compute = (most / k.per_cu) * round(k.per_cu) + round(most % k.per_cu) + more;
  return k.base + std::sqrt(compute * compute + memory * memory);
}

// the launches that read every tap from one window of consecutive pixels, if it fits
bool window_takes(const ConvGeom& g) {
  using D = Deep<2, 1, true>;
  return g.r == g.s && g.r * g.s >= 2 * D::KS - 1 && g.stride == 1 && 2 * g.pad == g.r - 1 && g.pad_dx == 0 &&
         g.p == g.h && g.q == g.wd && D::BM + 2 * (g.pad * g.wd + g.pad) <= D::WROWS;
}

// the fastest of the kernels in this file, and its prediction
int best_x3(const ConvGeom& g, long M, long K, double* us) {
  const bool window = window_takes(g);
  int best = -1;
  for (int v = 0; v < X3_KINDS; ++v) {
    if (v == X3_WINDOW && !window) continue;
    const double t = predicted_us(kKinds[v], g, M, K);
    if (best < 0 || t < *us) { best = v; *us = t; }
  }
  return best;
}
double fp32_us(const ConvGeom& g, long M, long K) {
  return predicted_us(kKinds[conv_igemm_two_groups(g, M, K) ? F32_TWO : F32_ONE], g, M, K);
}

// The same for the parts of a strided data gradient in one launch of a short kernel: the longest tile alone, or the compute
// units' share of all tiles and part of a last one.  These constants and those of conv_igemm_x3_parts_takes() are fitted to
// 45 shapes (2 to 256 images, 32 to 1024 channels, 3x3 and 5x5, stride 2), the sub-filters' launch included: median errors of
// 3 to 5 %, and on 73 shapes the choice is within 0.2 % of the best of the three ways on average, 5 % at most.
double predicted_parts_us(bool wide, const ConvGeom* parts, int n) {
  const Kind& k = kKinds[wide ? X3_128 : X3_64];
  double work = 0, longest = 0, last = 0;
  for (int i = 0; i < n; ++i) {
    const ConvGeom& g = parts[i];
    const long M = (long)g.n_img * g.p * g.q, steps = ((long)g.r * g.s * g.c + 15) / 16;
    const long tiles = ((M + k.bm - 1) / k.bm) * ((g.n_out + k.bn - 1) / k.bn);
    const double next = k.next + k.next_step * steps, first = k.first + k.first_step * steps;
    work += tiles * next;
    if (first > longest) longest = first;
    if (next > last) last = next;
  }
  const double share = work / 256 + last * (wide ? 0.51 : 0.27), alone = longest * (wide ? 0.965 : 1.12);
  return (wide ? 13.1 : 9.6) + 1.08 * (share > alone ? share : alone);
}

template <int MB, int NB>
void launch_parts(X3Parts& ps, int n, hipStream_t st, LaunchProbe* probe, long side_blocks) {
  probe->variant = V_IGEMM_X3;
  probe->kernel = MB == 2 ? "igemm_x3_parts 128x128" : "igemm_x3_parts 64x64";
  if (probe->dry) return;
  const int tn = (ps.g[0].n_out + 64 * NB - 1) / (64 * NB);
  long per_xcd = 0;
  for (int i = 0; i < n; ++i) {
    ps.tiles[i] = (ps.M[i] + 64 * MB - 1) / (64 * MB) * tn;
    ps.per_xcd[i] = (ps.tiles[i] + 7) / 8;
    per_xcd += ps.per_xcd[i];
  }
  const int main_grid = (int)(per_xcd * 8);
  if (probe->before) (void)hipEventRecord(probe->before, st);
  hipLaunchKernelGGL((igemm_x3_parts_kernel<MB, NB>), dim3((unsigned)(main_grid + side_blocks)), dim3(256), 0, st, ps, tn, main_grid);
  if (probe->after) (void)hipEventRecord(probe->after, st);
}

}  // namespace

bool conv_igemm_x3_takes(const ConvGeom& g, long M, long K) {
  // whole 16-channel steps inside one tap; a 1x1 filter may end inside a step (1000 classes: the fully connected layer's
  // data gradient at minibatch 41 49 us in the per-element kernel, 24 here)
  if (g.dtype != DT_F32 || g.c % (g.r * g.s == 1 ? 4 : 16) != 0 || g.c < 16 || g.r * g.s > 32) return false;
  // both operands within 32-bit byte ranges (the last bytes stay free for the offset that stands for
  // "outside"), 16-byte aligned
  const long margin_px = (long)g.pad * g.wd + g.pad + g.pad_dx;
  if ((margin_px + (long)g.n_img * g.h * g.wd) * g.c * 4 > 0xFFFFFF00L || (long)g.n_out * K * 4 > 0xFFFFFF00L) return false;
  if ((reinterpret_cast<uintptr_t>(g.in) & 15) || (reinterpret_cast<uintptr_t>(g.w) & 15)) return false;
  return ((M + 63) / 64) * ((g.n_out + 63) / 64) <= (1L << 30);
}

hipError_t conv_igemm_x3(const ConvGeom& g, int M, int K, hipStream_t st, LaunchProbe* probe) {
  if (g.side.count && (!g.side.part || !g.side.dw || g.side.splits < 1)) return hipErrorInvalidValue;
  if ((g.bias || g.relu) && (g.accumulate || g.stats || g.bnb.sums)) return hipErrorInvalidValue;
  const bool dense = g.out_stride == 1 && g.out_h == g.p && g.out_w == g.q;
  if (g.stats && (g.accumulate || !dense || conv_stat_slabs(M) > g.stats_stride)) return hipErrorInvalidValue;
  if (g.bnb.sums && (!g.bnb.x || !g.bnb.y || !g.bnb.mean || !g.bnb.istd || g.accumulate || !dense ||
                     conv_stat_slabs(M) > g.bnb.stride))
    return hipErrorInvalidValue;
  if (g.flip.wt && (!g.flip.w || g.flip.cout <= 0 || g.flip.cin <= 0 || g.flip.r <= 0 || g.flip.s <= 0)) return hipErrorInvalidValue;
  const long narrow = (long)((g.side.count + 1023) / 1024) + (g.flip.wt ? flip_tiles(g.flip.cout, g.flip.cin, g.flip.r, g.flip.s) : 0);
  const long tiles = (long)((M + 63) / 64) * ((g.n_out + 63) / 64);
  if (tiles + 8 + narrow > (1L << 30)) return hipErrorInvalidValue;
  double us = 0;
  const int best = best_x3(g, M, K, &us);
  switch (best) {
    case X3_128: launch_short<2, 2>(g, M, K, st, probe, narrow); break;
    case X3_64: launch_short<1, 1>(g, M, K, st, probe, narrow); break;
    case X3_WINDOW: launch_deep<2, 1, true>(g, M, K, st, probe); break;
    case X3_DEEP_2x1: launch_deep<2, 1, false>(g, M, K, st, probe); break;
    case X3_DEEP_2x2: launch_deep<2, 2, false>(g, M, K, st, probe); break;
    default: launch_deep<1, 1, false>(g, M, K, st, probe); break;
  }
  return probe->dry ? hipSuccess : hipGetLastError();
}

bool conv_igemm_x3_slower(const ConvGeom& g, long M, long K) {
  double us = 0;
  best_x3(g, M, K, &us);
  return fp32_us(g, M, K) < us * 1.02 + 0.3;
}

double conv_igemm_x3_us(const ConvGeom& g, long M, long K) {
  double us = 0;
  best_x3(g, M, K, &us);
  return g.c % 32 == 0 ? std::fmin(us, fp32_us(g, M, K)) : us;
}

// The parts go into one launch where that is predicted to take less than the parts one after the other: 128 channels of 56x56, 32
// images 93 -> 71 us, 512 of 14x14, 256 images 396 -> 350; not 1024 channels of 14x14, 64 images (366 us apart, 391 together) and
// 256 of 28x28 with 5x5 filters, 64 images (261, 276), which the deep kernels do better.
bool conv_igemm_x3_parts_takes(const ConvGeom* parts, int n) {
  if (n < 2 || n > kX3Parts) return false;
  double apart = 0;
  for (int i = 0; i < n; ++i) {
    const ConvGeom& g = parts[i];
    const long M = (long)g.n_img * g.p * g.q, K = (long)g.r * g.s * g.c;
    if (g.p <= 0 || g.q <= 0 || g.r <= 0 || g.s <= 0 || M >= (1L << 28) || K >= (1L << 31) || !conv_igemm_x3_takes(g, M, K)) return false;
    double us = 0;
    best_x3(g, M, K, &us);
    if (g.c % 32 == 0 && fp32_us(g, M, K) < us) us = fp32_us(g, M, K);
    apart += us;
  }
  const double a = predicted_parts_us(true, parts, n), b = predicted_parts_us(false, parts, n);
  return (a < b ? a : b) < 6.4 + 1.19 * apart;
}

hipError_t conv_igemm_x3_parts(const ConvGeom* parts, int n, hipStream_t st, LaunchProbe* probe) {
  const ConvGeom& g = parts[0];
  if (n < 1 || n > kX3Parts || !g.in || !g.out || g.n_img <= 0 || g.h <= 0 || g.wd <= 0 || (long)g.n_img * g.h * g.wd >= (1L << 31)) return hipErrorInvalidValue;
  if (g.side.count && (!g.side.part || !g.side.dw || g.side.splits < 1)) return hipErrorInvalidValue;
  if (g.flip.wt && (!g.flip.w || g.flip.cout <= 0 || g.flip.cin <= 0 || g.flip.r <= 0 || g.flip.s <= 0)) return hipErrorInvalidValue;
  int order[kX3Parts];
  for (int i = 0; i < n; ++i) {                   // the longest K first
    int j = i;
    for (; j > 0 && parts[order[j - 1]].r * parts[order[j - 1]].s < parts[i].r * parts[i].s; --j) order[j] = order[j - 1];
    order[j] = i;
  }
  X3Parts ps{};
  long tiles = 0;
  for (int i = 0; i < n; ++i) {
    const ConvGeom& c = parts[order[i]];
    if (!c.w || c.pad < 0 || c.pad + c.pad_dx < 0 || c.out_y0 < 0 || c.out_x0 < 0 ||
        c.out_y0 + (long)(c.p - 1) * c.out_stride >= c.out_h || c.out_x0 + (long)(c.q - 1) * c.out_stride >= c.out_w)
      return hipErrorInvalidValue;
    ps.g[i] = c;
    ps.M[i] = c.n_img * c.p * c.q;
    ps.K[i] = c.r * c.s * c.c;
    tiles += (long)((ps.M[i] + 63) / 64) * ((c.n_out + 63) / 64) + 8;
  }
  ps.g[0].side = g.side;                          // the side jobs are read from the first part of the launch
  ps.g[0].flip = g.flip;
  const long narrow = (long)((g.side.count + 1023) / 1024) + (g.flip.wt ? flip_tiles(g.flip.cout, g.flip.cin, g.flip.r, g.flip.s) : 0);
  if (tiles + narrow > (1L << 30)) return hipErrorInvalidValue;
  if (predicted_parts_us(true, parts, n) < predicted_parts_us(false, parts, n))
    launch_parts<2, 2>(ps, n, st, probe, narrow);
  else
    launch_parts<1, 1>(ps, n, st, probe, narrow);
  return probe->dry ? hipSuccess : hipGetLastError();
}

}  // namespace acc
