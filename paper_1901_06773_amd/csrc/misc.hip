// The small kernels that close the training step: filter flip/transposition for the data
// gradient, max-pooling, global average pooling, bias, softmax cross-entropy, SGD.
// None of them is on the roofline-critical path; all are coalesced along the channel
// axis of NHWC and use fixed-order reductions.
#include "kernels.h"
#include "dtype.h"
#include "dgrad_split.h"

namespace acc {
namespace {

constexpr int THREADS = 256;

inline unsigned grid_for(size_t work, size_t cap = 256 * 32) {
  size_t b = (work + THREADS - 1) / THREADS;
  if (b < 1) b = 1;
  return (unsigned)(b < cap ? b : cap);
}

// wt[ci][r'][t'][co] = w[co][R-1-r'][S-1-t'][ci]; a 32x32 LDS tile transposes (co, ci)
// so that both the read (ci fastest) and the write (co fastest) are coalesced.
// Bound by the launch and one trip to memory each way: a thread's four values are asked for at once, those that do not exist as the first.
template <class T>
__global__ __launch_bounds__(256) void flip_transpose_kernel(const T* __restrict__ w,
                                                             T* __restrict__ wt, int cout, int cin,
                                                             int r, int s) {
  __shared__ T tile[32][33];
  const int tap = blockIdx.z, taps = r * s;         // r'*s + t' of the output; flipped it is the last tap less that
  const int src_tap = taps - 1 - tap;
  const int co0 = blockIdx.y * 32, ci0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  T v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int co = co0 + ty + 8 * u, ci = ci0 + tx;
    v[u] = w[co < cout && ci < cin ? ((size_t)co * taps + src_tap) * cin + ci : 0];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) tile[ty + 8 * u][tx] = v[u];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int ci = ci0 + ty + 8 * u, co = co0 + tx;
    if (ci < cin && co < cout) wt[((size_t)ci * taps + tap) * cout + co] = tile[tx][ty + 8 * u];
  }
}

// wt[ci][r'][t'][co] = w[co][r0 + (nr-1-r')*step][t0 + (ns-1-t')*step][ci]: the sub-filters of all residue classes of a
// strided data gradient in one launch (a tap of w belongs to at most one of them; grid.z = taps); same tiling as above.
struct GatherParts {
  int r0[kMaxDgradParts], t0[kMaxDgradParts], nr[kMaxDgradParts], ns[kMaxDgradParts];
  size_t offset[kMaxDgradParts];
  int count;
};

template <class T>
__global__ __launch_bounds__(256) void gather_transpose_kernel(const T* __restrict__ w, char* __restrict__ out, int cout, int cin,
                                                               int r, int s, int step, GatherParts gp) {
  __shared__ T tile[32][33];
  const int co0 = blockIdx.y * 32, ci0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  for (int src_tap = blockIdx.z; src_tap < r * s; src_tap += gridDim.z) {
    const int kr = src_tap / s, kt = src_tap - kr * s;
    int part = -1, jr = 0, jt = 0;                  // the class of the tap, and the tap's place in it
    for (int i = 0; i < gp.count; ++i) {
      const int dr = kr - gp.r0[i], dt = kt - gp.t0[i], qr = dr / step, qt = dt / step;
      if (dr >= 0 && dt >= 0 && qr * step == dr && qt * step == dt && qr < gp.nr[i] && qt < gp.ns[i]) {
        part = i; jr = qr; jt = qt;
      }
    }
    if (part < 0) continue;                         // (the same for the whole workgroup)
    const int nr = gp.nr[part], ns = gp.ns[part], tap = (nr - 1 - jr) * ns + (ns - 1 - jt);
    T* wt = reinterpret_cast<T*>(out + gp.offset[part]);
    __syncthreads();
    T v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int co = co0 + ty + 8 * u, ci = ci0 + tx;
      v[u] = w[co < cout && ci < cin ? ((size_t)co * r * s + src_tap) * cin + ci : 0];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) tile[ty + 8 * u][tx] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int ci = ci0 + ty + 8 * u, co = co0 + tx;
      if (ci < cin && co < cout) wt[((size_t)ci * nr * ns + tap) * cout + co] = tile[tx][ty + 8 * u];
    }
  }
}

// one thread per (n, p, q, 4 channels); the first maximum in (r, t) scan order wins
template <class T>
__global__ __launch_bounds__(THREADS) void maxpool_fwd_kernel(const T* __restrict__ x,
                                                              T* __restrict__ y, int n, int h, int wd,
                                                              int c, int r, int s, int stride, int pad,
                                                              int ho, int wo) {
  const int cg = c >> 2;
  const size_t total = (size_t)n * ho * wo * cg;
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    const int g = (int)(i % cg);
    size_t rest = i / cg;
    const int q = (int)(rest % wo); rest /= wo;
    const int p = (int)(rest % ho);
    const int img = (int)(rest / ho);
    float best[4] = {0.f, 0.f, 0.f, 0.f};
    bool have = false;
    for (int kr = 0; kr < r; ++kr) {
      const int iy = p * stride + kr - pad;
      if ((unsigned)iy >= (unsigned)h) continue;
      for (int kt = 0; kt < s; ++kt) {
        const int ix = q * stride + kt - pad;
        if ((unsigned)ix >= (unsigned)wd) continue;
        float v[4];
        Elem<T>::load4(x + ((size_t)(img * h + iy) * wd + ix) * c + g * 4, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) best[j] = (!have || v[j] > best[j]) ? v[j] : best[j];
        have = true;
      }
    }
    Elem<T>::store4(y + i * 4, best);
  }
}

// The same for 3x3 windows, V channels (16 bytes) per thread: the nine loads go out together, places that do not exist read the nearest one
// that does and are not compared; indices in 32 bits.  Bound by HBM.  3x3/2 of 64 channels at 112x112: fp32, 32 images 31.6 -> 27.8 us
// (129 MB), 2 images 7.0 -> 4.2; bf16, 128 images 91.5 -> 50.1.
template <class T, int V>
__global__ __launch_bounds__(THREADS) void maxpool3_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, int total, int h, int wd, int c,
                                                               int stride, int pad, int ho, int wo) {
  const int cg = c / V;
  for (int i = blockIdx.x * THREADS + threadIdx.x; i < total; i += gridDim.x * THREADS) {
    const uint32_t pix = (uint32_t)i / (uint32_t)cg, g = i - pix * cg, row = pix / (uint32_t)wo, q = pix - row * wo;
    const uint32_t img = row / (uint32_t)ho, p = row - img * ho;
    const int iy = (int)p * stride - pad, ix = (int)q * stride - pad;
    const T* xi = x + (size_t)img * h * wd * c + (size_t)g * V;
    union Raw { uint4 u; T t[16 / sizeof(T)]; } v[9];
    bool ok[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int yy = iy + k / 3, xx = ix + k % 3;
      ok[k] = ((unsigned)yy < (unsigned)h) & ((unsigned)xx < (unsigned)wd);
      v[k].u = *reinterpret_cast<const uint4*>(xi + ((size_t)min(max(yy, 0), h - 1) * wd + min(max(xx, 0), wd - 1)) * c);
    }
    Raw best = v[0];
    bool have = false;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const bool more = ok[k] & (!have | (Elem<T>::load(&v[k].t[j]) > Elem<T>::load(&best.t[j])));
        best.t[j] = more ? v[k].t[j] : best.t[j];
      }
      have |= ok[k];
    }
    *reinterpret_cast<uint4*>(y + (size_t)i * V) = best.u;
  }
}

// Gather form of the max-pool gradient: one thread per input position and group of V
// channels (V = 4 as float4 when c % 4 == 0, else 1); for every window that covers the
// position, find the window's first maximum again and take the window's dy where this
// position is the winner.  Windows are visited in (p, q) order, so the sum has a fixed order.
template <class T, int V>
__global__ __launch_bounds__(THREADS) void maxpool_bwd_kernel(const T* __restrict__ x,
                                                              const T* __restrict__ dy, T* dx,
                                                              int n, int h, int wd, int c, int r, int s,
                                                              int stride, int pad, int ho, int wo,
                                                              int accumulate) {
  struct Vec { float v[V]; };
  auto ld = [](const T* p) { Vec r; if constexpr (V == 4) Elem<T>::load4(p, r.v); else r.v[0] = Elem<T>::load(p); return r; };
  auto st = [](T* p, const Vec& r) { if constexpr (V == 4) Elem<T>::store4(p, r.v); else Elem<T>::store(p, r.v[0]); };
  const int cg = c / V;
  const size_t total = (size_t)n * h * wd * cg;
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    const int g = (int)(i % cg);
    size_t rest = i / cg;
    const int ix = (int)(rest % wd); rest /= wd;
    const int iy = (int)(rest % h);
    const int img = (int)(rest / h);
    const int me = iy * wd + ix;
    // windows p with p*stride - pad <= iy <= p*stride - pad + r - 1
    int p_lo = (iy + pad - r + 1 + stride - 1);
    p_lo = p_lo > 0 ? p_lo / stride : 0;
    int p_hi = (iy + pad) / stride; if (p_hi > ho - 1) p_hi = ho - 1;
    int q_lo = (ix + pad - s + 1 + stride - 1);
    q_lo = q_lo > 0 ? q_lo / stride : 0;
    int q_hi = (ix + pad) / stride; if (q_hi > wo - 1) q_hi = wo - 1;
    Vec acc;
#pragma unroll
    for (int j = 0; j < V; ++j) acc.v[j] = 0.f;
    for (int p = p_lo; p <= p_hi; ++p)
      for (int q = q_lo; q <= q_hi; ++q) {
        Vec best;
        int at[V];
#pragma unroll
        for (int j = 0; j < V; ++j) { best.v[j] = 0.f; at[j] = -1; }
        for (int kr = 0; kr < r; ++kr) {
          const int yy = p * stride + kr - pad;
          if ((unsigned)yy >= (unsigned)h) continue;
          for (int kt = 0; kt < s; ++kt) {
            const int xx = q * stride + kt - pad;
            if ((unsigned)xx >= (unsigned)wd) continue;
            const Vec v = ld(x + ((size_t)(img * h + yy) * wd + xx) * c + g * V);
#pragma unroll
            for (int j = 0; j < V; ++j)
              if (at[j] < 0 || v.v[j] > best.v[j]) { best.v[j] = v.v[j]; at[j] = yy * wd + xx; }
          }
        }
        const Vec d = ld(dy + ((size_t)(img * ho + p) * wo + q) * c + g * V);
#pragma unroll
        for (int j = 0; j < V; ++j)
          if (at[j] == me) acc.v[j] += d.v[j];
      }
    T* out = dx + i * V;
    if (accumulate) {
      const Vec o = ld(out);
#pragma unroll
      for (int j = 0; j < V; ++j) acc.v[j] = o.v[j] + acc.v[j];
    }
    st(out, acc);
  }
}

// The same for 3x3 windows at stride 2 with padding 1 (the stem pool of the ResNets): one thread
// per column of 2x2 blocks of input positions (`strip` of them, top to bottom) and four channels.  The block (rows
// 2a, 2a+1, columns 2b, 2b+1) is covered by the windows p in {a, a+1}, q in {b, b+1} and by no other.  Going down, the
// windows of row a+1 are the next block's row a, and their first input row is the last one of the windows above: ten
// loads of x per block where every block on its own takes 36 (64 channels, 112x112, 32 images: 103 us a block at a time in
// the kernel before, 48 now; the 232 MB it has to move take 50 at the rate of a large copy).  Windows are visited in the same (p, q) order and the same
// first maximum wins, so every sum has the same terms in the same order as in the kernel above.
//
// Longer strips load less and leave fewer threads, each a longer chain of trips to memory.  Measured at strips of 1 / 2 / 4 / 8
// (and the kernel before), 64 channels: fp32, 2 images of 112x112 (100 thousand blocks) 7.7 / 9.0 / 14.4 / 22.9 (11.5) us; 4 images
// (200 thousand) 12.9 / 11.8 / 15.5 / 25.1 (18.8); 16 images (0.8 million) 37 / 31 / 28 / 31 (52); 32 images 66 / 54 / 49.5 /
// 47.9 (103); bf16 at 32 images, by a scan, 62 / 49 / 45 / 50 (75).
inline int maxpool_strip(size_t blocks, size_t elem_bytes) {
  if (blocks < 160 << 10) return 1;
  if (blocks < 512 << 10) return 2;
  return elem_bytes == 2 || blocks < 1280 << 10 ? 4 : 8;
}
// Three rows of five columns of x, four channels each, and in every 3x3 window over them the first position that holds the
// maximum.  NaN as in a plain scan with ">": at the first position of a window (that lies in the map) it stays, elsewhere it
// is passed over.
template <class T> struct FirstMax;
template <> struct FirstMax<float> {
  float v[3][5][4];
  bool row_ok[3], col_ok[5];
  __device__ __forceinline__ void load(int i, const float* p, int c, const int (&col)[5], const bool (&cols)[5], bool ok) {
    row_ok[i] = ok;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      col_ok[t] = cols[t];
      Elem<float>::load4(p + (size_t)col[t] * c, v[i][t]);
    }
  }
  __device__ __forceinline__ void down() {
    row_ok[0] = row_ok[2];
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[0][t][j] = v[2][t][j];
  }
  __device__ __forceinline__ void head(int, const bool (&)[5]) {}
  static __device__ __forceinline__ int place(int at, int) { return at; }      // 3 * row + column
  __device__ __forceinline__ void first(int (&at)[4], int t0) const {
    float best[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) at[j] = -1;
#pragma unroll
    for (int kr = 0; kr < 3; ++kr)
#pragma unroll
      for (int kt = 0; kt < 3; ++kt) {
        const bool ok = row_ok[kr] && col_ok[t0 + kt];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float x = v[kr][t0 + kt][j];
          const bool more = ok & ((at[j] < 0) | (x > best[j]));
          best[j] = more ? x : best[j];
          at[j] = more ? 3 * kr + kt : at[j];
        }
      }
  }
};
// bf16: an integer per value, its rank (16 bits that compare as the values do: both zeros are one, a NaN and what lies outside
// the map rank below everything) above a number that falls from 15 to 1 along the three rows of five.  The largest integer of
// a window is its first maximum, and a row can be left as the largest of its part of either window: eight registers in place
// of twenty, and two instructions for a value of a row and its windows where the scan has five for each value of a window.
// Registers decide here: with all fifteen integers kept and a scan for rows that hold a NaN (147 to 170 registers, three or two
// waves instead of four) the kernel took 288 to 370 us.  64 channels of 112x112, scan and this, 2 / 8 / 32 / 128 images: 7.8 / 18.6 /
// 45.8 / 168 and 7.4 / 15.8 / 38.5 / 153 us (the 514 MB of 128 images take 111 at the rate of a large copy); what is left
// is the loads of overlapping columns and the wait for them.
template <> struct FirstMax<bf16_t> {
  typedef short Short2 __attribute__((ext_vector_type(2)));
  typedef unsigned short UShort2 __attribute__((ext_vector_type(2)));
  int key[3][2][4];
  unsigned lead[3][2][2];                         // the first values of either part, as loaded
  static __device__ __forceinline__ unsigned bits(Short2 v) { return __builtin_bit_cast(unsigned, v); }
  __device__ __forceinline__ void load(int i, const bf16_t* p, int c, const int (&col)[5], const bool (&cols)[5], bool ok) {
    uint2 q[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) q[t] = *reinterpret_cast<const uint2*>(p + (size_t)col[t] * c);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      int v[5][2];
#pragma unroll
      for (int t = 0; t < 5; ++t) {
        const unsigned w = k ? q[t].y : q[t].x;
        const Short2 sign = __builtin_bit_cast(Short2, w) >> 15;
        // negative values downwards from zero; 127 more, which takes a positive NaN round to the lowest
        const Short2 r = __builtin_bit_cast(Short2, w ^ (bits(sign) & 0x7fff7fffu)) - sign + (short)0x7f;
        const unsigned rank = ok && cols[t] ? bits(r) : 0x80008000u, code = 15 - (5 * i + t);
        v[t][0] = (int)(rank << 16 | code);
        v[t][1] = (int)((rank & 0xffff0000u) | code);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        key[i][0][2 * k + j] = max(max(v[0][j], v[1][j]), v[2][j]);
        key[i][1][2 * k + j] = max(max(v[2][j], v[3][j]), v[4][j]);
      }
      lead[i][0][k] = cols[0] ? (k ? q[0].y : q[0].x) : (k ? q[1].y : q[1].x);
      lead[i][1][k] = k ? q[2].y : q[2].x;
    }
  }
  __device__ __forceinline__ void down() {
#pragma unroll
    for (int w = 0; w < 2; ++w) {
#pragma unroll
      for (int j = 0; j < 4; ++j) key[0][w][j] = key[2][w][j] + 10;
      lead[0][w][0] = lead[2][w][0];
      lead[0][w][1] = lead[2][w][1];
    }
  }
  // row i is the first one of its windows: a NaN at their first position stays
  __device__ __forceinline__ void head(int i, const bool (&cols)[5]) {
    UShort2 top = 0;
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int k = 0; k < 2; ++k) top = __builtin_elementwise_max(top, __builtin_bit_cast(UShort2, lead[i][w][k] & 0x7fff7fffu));
    if (top.x <= 0x7f80 && top.y <= 0x7f80) return;
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((lead[i][w][j >> 1] >> 16 * (j & 1) & 0x7fffu) > 0x7f80u)
          key[i][w][j] = 0x7fff0000 | (15 - (5 * i + (w ? 2 : cols[0] ? 0 : 1)));
  }
  static __device__ __forceinline__ int place(int at, int t0) { return 15 - (5 * (at / 3) + at % 3 + t0); }
  __device__ __forceinline__ void first(int (&at)[4], int t0) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) at[j] = max(max(key[0][t0 >> 1][j], key[1][t0 >> 1][j]), key[2][t0 >> 1][j]) & 15;
  }
};
template <class T>
__global__ __launch_bounds__(THREADS) void maxpool3s2_bwd_kernel(const T* __restrict__ x,
                                                                 const T* __restrict__ dy, T* __restrict__ dx, int n,
                                                                 int h, int wd, int c, int ho, int wo,
                                                                 int accumulate, int strip) {
  const int cg = c >> 2, hb = (h + 1) >> 1, wb = (wd + 1) >> 1, strips = (hb + strip - 1) / strip;
  const size_t total = (size_t)n * strips * wb * cg;
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    const int g = (int)(i % cg);
    size_t rest = i / cg;
    const int b = (int)(rest % wb); rest /= wb;
    const int a0 = (int)(rest % strips) * strip;
    const int img = (int)(rest / strips);
    const T* xi = x + (size_t)img * h * wd * c + g * 4;
    const T* dyi = dy + (size_t)img * ho * wo * c + g * 4;
    T* dxi = dx + (size_t)img * h * wd * c + g * 4;
    bool col_ok[5];
    int col[5];
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      const int xx = 2 * b - 1 + t;
      col_ok[t] = (unsigned)xx < (unsigned)wd;
      col[t] = col_ok[t] ? xx : 0;
    }
    FirstMax<T> rows;                            // three rows of x and the windows over them
    struct Win { int at[4]; float d[4]; };       // which position holds the first maximum, gradient of the window
    auto load_row = [&](int i, int yy) {
      const bool ok = (unsigned)yy < (unsigned)h;
      const T* p = xi + (size_t)(ok ? yy : 0) * wd * c;
      rows.load(i, p, c, col, col_ok, ok);
    };
    auto window = [&](Win& w, int p, int q, int t0) {
      const bool exists = p < ho && q < wo;
      rows.first(w.at, t0);
      Elem<T>::load4(dyi + (exists ? ((size_t)p * wo + q) * c : 0), w.d);
#pragma unroll
      for (int j = 0; j < 4; ++j) w.at[j] = exists ? w.at[j] : -1;
    };
    Win u0, u1, l0, l1;                          // windows (a, b), (a, b+1) and (a+1, b), (a+1, b+1)
    load_row(0, 2 * a0 - 1);
    load_row(1, 2 * a0);
    load_row(2, 2 * a0 + 1);
    if (a0 == 0) rows.head(1, col_ok);
    else rows.head(0, col_ok);
    window(u0, a0, b, 0);
    window(u1, a0, b + 1, 2);
    for (int a = a0; a < a0 + strip && a < hb; ++a) {
      rows.down();
      load_row(1, 2 * a + 2);
      load_row(2, 2 * a + 3);
      rows.head(0, col_ok);
      window(l0, a + 1, b, 0);
      window(l1, a + 1, b + 1, 2);
      float o[2][2][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        auto take = [&](float acc, const Win& w, int at, int t0) { return w.at[j] == FirstMax<T>::place(at, t0) ? acc + w.d[j] : acc; };
        o[0][0][j] = take(0.f, u0, 4, 0);
        o[0][1][j] = take(take(0.f, u0, 5, 0), u1, 3, 2);
        o[1][0][j] = take(take(0.f, u0, 7, 0), l0, 1, 0);
        o[1][1][j] = take(take(take(take(0.f, u0, 8, 0), u1, 6, 2), l0, 2, 0), l1, 0, 2);
      }
#pragma unroll
      for (int ry = 0; ry < 2; ++ry)
#pragma unroll
        for (int rx = 0; rx < 2; ++rx) {
          const int iy = 2 * a + ry, ix = 2 * b + rx;
          if (iy >= h || ix >= wd) continue;
          T* out = dxi + ((size_t)iy * wd + ix) * c;
          if (accumulate) {
            float old[4];
            Elem<T>::load4(out, old);
#pragma unroll
            for (int j = 0; j < 4; ++j) o[ry][rx][j] = old[j] + o[ry][rx][j];
          }
          Elem<T>::store4(out, o[ry][rx]);
        }
      u0 = l0;
      u1 = l1;
    }
  }
}

// Workgroups along the images of the two kernels below at most; they walk on from there (a launch may have fewer than 2^32
// threads in a dimension).
constexpr int kGapImages = 1 << 20;

// y[n][c] = mean over hw of x[n][hw][c].  A workgroup takes one image at a time and up to 256 channels: tpr threads of four
// channels each across a row, the other threads further rows (four in flight each); the row groups are added in order.
// (One thread per channel and image, all rows one after the other, waited for every row in turn: 2 x 64 channels of
// 16x16 67 us, 41 x 2048 of 7x7 16.5 us; now 5 and 6.)
template <class T>
__global__ __launch_bounds__(THREADS) void gap_fwd4_kernel(const T* __restrict__ x, T* __restrict__ y, int n, int hw, int c, int tpr, int rpi) {
  __shared__ float red[THREADS][4];
  const int tid = threadIdx.x, lane_r = tid / tpr, lane_c = tid - lane_r * tpr;
  const int ch = (blockIdx.y * tpr + lane_c) * 4;
  const bool active = lane_r < rpi && ch < c;
  for (int img = blockIdx.x; img < n; img += gridDim.x) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (active) {
      const T* p = x + (size_t)img * hw * c + ch;
      int k = lane_r;
      for (; k + 3 * rpi < hw; k += 4 * rpi) {
        float v[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) Elem<T>::load4(p + (size_t)(k + u * rpi) * c, v[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) s[j] += v[u][j];
      }
      for (; k < hw; k += rpi) {
        float v[4];
        Elem<T>::load4(p + (size_t)k * c, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += v[j];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) red[tid][j] = s[j];
    __syncthreads();
    if (lane_r == 0 && active) {
      for (int r = 1; r < rpi; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += red[r * tpr + lane_c][j];
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] = s[j] / (float)hw;
      Elem<T>::store4(y + (size_t)img * c + ch, s);
    }
    __syncthreads();                                   // the sums are no longer read
  }
}

// the same for channel counts or addresses that do not allow four channels at a time
template <class T>
__global__ __launch_bounds__(THREADS) void gap_fwd_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                          int n, int hw, int c) {
  const size_t total = (size_t)n * c;
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    const int ch = (int)(i % c);
    const int img = (int)(i / c);
    float sum = 0.f;
    for (int k = 0; k < hw; ++k) sum += Elem<T>::load(x + ((size_t)img * hw + k) * c + ch);
    Elem<T>::store(y + i, sum / (float)hw);
  }
}

// dx[n][k][c] (+)= dy[n][c] / hw; four channels per thread, rows as in gap_fwd4_kernel, blockIdx.z a range of them
template <class T>
__global__ __launch_bounds__(THREADS) void gap_bwd4_kernel(const T* __restrict__ dy, T* __restrict__ dx, int n, int hw, int c, int tpr, int rpi,
                                                           int rows_per_block, int accumulate) {
  const int tid = threadIdx.x, lane_r = tid / tpr, lane_c = tid - lane_r * tpr;
  const int ch = (blockIdx.y * tpr + lane_c) * 4;
  if (lane_r >= rpi || ch >= c) return;
  const float inv = 1.f / (float)hw;
  const int lo = blockIdx.z * rows_per_block, hi = lo + rows_per_block < hw ? lo + rows_per_block : hw;
  for (int img = blockIdx.x; img < n; img += gridDim.x) {
    float v[4];
    Elem<T>::load4(dy + (size_t)img * c + ch, v);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] *= inv;
    T* p = dx + (size_t)img * hw * c + ch;
    for (int k = lo + lane_r; k < hi; k += rpi) {
      if (accumulate) {
        float o[4];
        Elem<T>::load4(p + (size_t)k * c, o);
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] += v[j];
        Elem<T>::store4(p + (size_t)k * c, o);
      } else {
        Elem<T>::store4(p + (size_t)k * c, v);
      }
    }
  }
}

template <class T>
__global__ __launch_bounds__(THREADS) void gap_bwd_kernel(const T* __restrict__ dy, T* dx, int n,
                                                          int hw, int c, int accumulate) {
  const size_t total = (size_t)n * hw * c;
  const float inv = 1.f / (float)hw;
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    const int ch = (int)(i % c);
    const int img = (int)(i / ((size_t)hw * c));
    const float v = Elem<T>::load(dy + (size_t)img * c + ch) * inv;
    Elem<T>::store(dx + i, accumulate ? Elem<T>::load(dx + i) + v : v);
  }
}

template <class T>
__global__ __launch_bounds__(THREADS) void bias_add_kernel(T* y, const float* __restrict__ b, size_t total,
                                                           int c, int relu) {
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    float v = Elem<T>::load(y + i) + b[i % c];
    if (relu) v = fmaxf(v, 0.f);
    Elem<T>::store(y + i, v);
  }
}

// Backward of y = relu(x + b): a workgroup takes one slab of rows and up to 256 channels (four
// per thread), writes g = dy * [y > 0] over dy and the per-channel sums of g over its slab to
// part[slab][c]; rows of a slab are spread over the threads that share a channel group and
// added in a fixed order.  The second kernel adds the slabs in order.
constexpr int RB_MAX_SLABS = 512;
template <class T>
__global__ __launch_bounds__(THREADS) void relu_bias_bwd_kernel(T* dy, const T* __restrict__ y,
                                                                double* __restrict__ part, long rows, int c,
                                                                int tpr, int rpi, long rows_per_slab) {
  __shared__ double red[THREADS][4];
  const int tid = threadIdx.x;
  const int lane_r = tid / tpr, lane_c = tid - lane_r * tpr;
  const int cg = blockIdx.y * tpr + lane_c;
  const bool active = lane_r < rpi && cg * 4 < c;
  const long r_lo = (long)blockIdx.x * rows_per_slab;
  const long r_hi = r_lo + rows_per_slab < rows ? r_lo + rows_per_slab : rows;
  double s[4] = {0, 0, 0, 0};
  if (active)
    for (long r = r_lo + lane_r; r < r_hi; r += rpi) {
      const size_t off = (size_t)r * c + (size_t)cg * 4;
      float gv[4];
      Elem<T>::load4(dy + off, gv);
      if (y) {
        float yv[4];
        Elem<T>::load4(y + off, yv);
#pragma unroll
        for (int j = 0; j < 4; ++j) gv[j] = yv[j] > 0.f ? gv[j] : 0.f;
        Elem<T>::store4(dy + off, gv);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] += (double)gv[j];
    }
#pragma unroll
  for (int j = 0; j < 4; ++j) red[tid][j] = s[j];
  __syncthreads();
  if (lane_r == 0 && cg * 4 < c) {
    for (int rr = 1; rr < rpi; ++rr)
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] += red[rr * tpr + lane_c][j];
#pragma unroll
    for (int j = 0; j < 4; ++j) part[(size_t)blockIdx.x * c + (size_t)cg * 4 + j] = s[j];
  }
}

template <class T>
__global__ __launch_bounds__(THREADS) void relu_mask_kernel(T* dy, const T* __restrict__ y, size_t count) {
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < count; i += (size_t)gridDim.x * THREADS)
    if (!(Elem<T>::load(y + i) > 0.f)) Elem<T>::store(dy + i, 0.f);
}

__global__ __launch_bounds__(THREADS) void slab_sum_kernel(const double* __restrict__ part, float* __restrict__ db,
                                                           int slabs, int c) {
  const int ch = blockIdx.x * THREADS + threadIdx.x;
  if (ch >= c) return;
  double sum = 0.0;
  for (int k = 0; k < slabs; ++k) sum += part[(size_t)k * c + ch];
  db[ch] = (float)sum;
}

// db[ch] = sum over rows, one thread per channel, rows in order
template <class T>
__global__ __launch_bounds__(THREADS) void column_sum_kernel(const T* __restrict__ dy,
                                                             float* __restrict__ db, long rows, int c) {
  const int ch = blockIdx.x * THREADS + threadIdx.x;
  if (ch >= c) return;
  float sum = 0.f;
  long r = 0;
  for (; r + 16 <= rows; r += 16) {     // sixteen rows on their way at once
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = Elem<T>::load(dy + (size_t)(r + u) * c + ch);
#pragma unroll
    for (int u = 0; u < 16; ++u) sum += v[u];
  }
  for (; r < rows; ++r) sum += Elem<T>::load(dy + (size_t)r * c + ch);
  db[ch] = sum;
}

// Fixed-order block reductions: a butterfly in every wave, then the waves in order.
template <class F>
__device__ __forceinline__ float block_reduce(float v, float* sh, F op) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = sh[0];
#pragma unroll
  for (int w = 1; w < THREADS / 64; ++w) r = op(r, sh[w]);
  __syncthreads();
  return r;
}

// one workgroup per sample: loss_rows[i] = logsumexp(z_i) - z_i[label]; optionally
// dz = (softmax - onehot) / n.  V > 0: at most V * THREADS classes, a thread keeps its logits.
// Bound by the launch and trips through LDS: 41 rows of 1000 classes, loss and gradient 13 us in three launches, 9 in two.
template <class T, int V>
__global__ __launch_bounds__(THREADS) void softmax_ce_kernel(const T* __restrict__ z,
                                                             const int32_t* __restrict__ labels,
                                                             float* __restrict__ loss_rows,
                                                             T* __restrict__ dz, int n, int classes) {
  __shared__ float sh[THREADS / 64];
  const int i = blockIdx.x;
  const T* zi = z + (size_t)i * classes;
  const int lab = labels[i];
  // a label outside [0, classes) reads nothing: the row's loss is NaN and its gradient has no one-hot term
  const bool lab_ok = (unsigned)lab < (unsigned)classes;
  float z_lab = Elem<T>::load(zi + (lab_ok ? lab : 0));
  asm volatile("" : "+v"(z_lab));      // read here: dz may be z, and another thread's gradient lies there later
  float v[V > 0 ? V : 1];
  auto each = [&](auto&& use) {
    if constexpr (V > 0) {
#pragma unroll
      for (int u = 0; u < V; ++u)
        if ((int)threadIdx.x + u * THREADS < classes) use((int)threadIdx.x + u * THREADS, v[u]);
    } else {
      for (int j = threadIdx.x; j < classes; j += THREADS) use(j, Elem<T>::load(zi + j));
    }
  };
  if constexpr (V > 0) {
#pragma unroll
    for (int u = 0; u < V; ++u) v[u] = Elem<T>::load(zi + min((int)threadIdx.x + u * THREADS, classes - 1));
  }
  float mx = -INFINITY;
  each([&](int, float t) { mx = fmaxf(mx, t); });
  mx = block_reduce(mx, sh, [](float a, float b) { return fmaxf(a, b); });
  float se = 0.f;
  each([&](int, float t) { se += expf(t - mx); });
  se = block_reduce(se, sh, [](float a, float b) { return a + b; });
  // everything relative to the row maximum: z - mx is exact for the logits near the maximum (the only ones
  // that matter), so neither the loss nor a probability close to one loses digits to the size of the logits
  const float lg = logf(se);
  if (loss_rows && threadIdx.x == 0) loss_rows[i] = lab_ok ? lg - (z_lab - mx) : NAN;
  if (dz) {
    const float inv_n = 1.f / (float)n;
    each([&](int j, float t) {
      Elem<T>::store(dz + (size_t)i * classes + j, (expf((t - mx) - lg) - (j == lab ? 1.f : 0.f)) * inv_n);
    });
  }
}

// loss = (1/n) * sum of rows, added in index order by one wave-sized loop
__global__ void loss_mean_kernel(const float* __restrict__ loss_rows, float* __restrict__ loss, int n) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double s = 0.0;
    int i = 0;
    for (; i + 16 <= n; i += 16) {      // sixteen on their way at once
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = loss_rows[i + u];
#pragma unroll
      for (int u = 0; u < 16; ++u) s += (double)v[u];
    }
    for (; i < n; ++i) s += (double)loss_rows[i];
    *loss = (float)(s / n);
  }
}

// w <- w - lr * g on the fp32 master weights; in bf16 mode the rounded copy the kernels read is
// refreshed in the same pass
__global__ __launch_bounds__(THREADS) void sgd_kernel(float* __restrict__ w, const float* __restrict__ g,
                                                      float lr, size_t count, bf16_t* __restrict__ w16) {
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < count; i += (size_t)gridDim.x * THREADS) {
    const float v = fmaf(-lr, g[i], w[i]);
    w[i] = v;
    if (w16) w16[i] = float_to_bf16(v);
  }
}

__global__ __launch_bounds__(THREADS) void fill_zero_kernel(float* __restrict__ p, size_t count) {
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < count; i += (size_t)gridDim.x * THREADS)
    p[i] = 0.f;
}

// y[n][hw][c] = x[n][c][hw]: reads coalesced along hw for each channel, one pixel per thread (few channels)
template <class T>
__global__ __launch_bounds__(THREADS) void nchw_to_nhwc_kernel(const float* __restrict__ x, T* __restrict__ y,
                                                               int n, int c, int hw) {
  const size_t total = (size_t)n * hw;
  for (size_t i = (size_t)blockIdx.x * THREADS + threadIdx.x; i < total; i += (size_t)gridDim.x * THREADS) {
    const size_t img = i / hw, pos = i - img * hw;
    const float* src = x + img * (size_t)c * hw + pos;
    T* dst = y + i * c;
    for (int ch = 0; ch < c; ++ch) Elem<T>::store(dst + ch, src[(size_t)ch * hw]);
  }
}

// many channels: 32 x 32 (channel, pixel) tiles through LDS, both sides coalesced (64 channels, 2 x 16x16 pixels: 22.8
// -> 4 us, where a thread of the kernel above reads 64 values one after the other)
template <class T>
__global__ __launch_bounds__(THREADS) void nchw_to_nhwc_tile_kernel(const float* __restrict__ x, T* __restrict__ y,
                                                                    int c, int hw, int tiles_p, int tiles_c) {
  __shared__ float tile[32][33];
  const int tp = blockIdx.x % tiles_p, rest = blockIdx.x / tiles_p, tc = rest % tiles_c, img = rest / tiles_c;
  const int p0 = tp * 32, c0 = tc * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const float* src = x + (size_t)img * c * hw;
  for (int i = ty; i < 32; i += 8) tile[i][tx] = c0 + i < c && p0 + tx < hw ? src[(size_t)(c0 + i) * hw + p0 + tx] : 0.f;
  __syncthreads();
  T* dst = y + (size_t)img * c * hw;
  for (int i = ty; i < 32; i += 8)
    if (p0 + i < hw && c0 + tx < c) Elem<T>::store(dst + (size_t)(p0 + i) * c + c0 + tx, tile[tx][i]);
}

}  // namespace

// runs `call` with T = float or bf16_t according to dtype
#define ACC_DISPATCH(dtype, call)                                   \
  do {                                                              \
    if ((dtype) == DT_F32) { using T = float; call; }               \
    else if ((dtype) == DT_BF16) { using T = bf16_t; call; }        \
    else return hipErrorInvalidValue;                               \
  } while (0)

hipError_t nchw_to_nhwc(const float* x, void* y, int n, int c, int hw, int dtype, hipStream_t st) {
  if (!x || !y || n <= 0 || c <= 0 || hw <= 0) return hipErrorInvalidValue;
  const long tiles_p = (hw + 31L) / 32, tiles_c = (c + 31L) / 32;
  if (c >= 8 && tiles_p * tiles_c * n < (1L << 24)) {        // (a launch has fewer than 2^32 threads)
    ACC_DISPATCH(dtype, hipLaunchKernelGGL(nchw_to_nhwc_tile_kernel<T>, dim3((unsigned)(tiles_p * tiles_c * n)), dim3(THREADS), 0, st,
                                           x, (T*)y, c, hw, (int)tiles_p, (int)tiles_c));
    return hipGetLastError();
  }
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(nchw_to_nhwc_kernel<T>, dim3(grid_for((size_t)n * hw)), dim3(THREADS), 0, st,
                                         x, (T*)y, n, c, hw));
  return hipGetLastError();
}

hipError_t filter_flip_transpose(const void* w, void* wt, int cout, int cin, int r, int s, int dtype,
                                 hipStream_t st) {
  if (!w || !wt || cout <= 0 || cin <= 0 || r <= 0 || s <= 0 || r * s > 65535) return hipErrorInvalidValue;
  const dim3 grid((cin + 31) / 32, (cout + 31) / 32, r * s);
  if (grid.y > 65535) return hipErrorInvalidValue;
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(flip_transpose_kernel<T>, grid, dim3(256), 0, st, (const T*)w, (T*)wt, cout,
                                         cin, r, s));
  return hipGetLastError();
}

hipError_t filter_gather_transpose(const DgradSplit& d, void* wt, int dtype, hipStream_t st) {
  if (!d.w || !wt || !d.parts || d.count <= 0 || d.count > kMaxDgradParts || d.cout <= 0 || d.cin <= 0 || d.r <= 0 || d.s <= 0 ||
      d.stride <= 0 || (long)d.r * d.s >= (1L << 31))
    return hipErrorInvalidValue;
  GatherParts gp{};
  gp.count = d.count;
  for (int i = 0; i < d.count; ++i) {
    const DgradPart& pt = d.parts[i];
    if (pt.nr <= 0 || pt.ns <= 0 || pt.r0 < 0 || pt.t0 < 0 || pt.r0 + (pt.nr - 1) * d.stride >= d.r ||
        pt.t0 + (pt.ns - 1) * d.stride >= d.s)
      return hipErrorInvalidValue;
    gp.r0[i] = pt.r0; gp.t0[i] = pt.t0; gp.nr[i] = pt.nr; gp.ns[i] = pt.ns; gp.offset[i] = pt.wt_offset;
  }
  const dim3 grid((d.cin + 31) / 32, (d.cout + 31) / 32, d.r * d.s < 65535 ? d.r * d.s : 65535);
  if (grid.y > 65535) return hipErrorInvalidValue;
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(gather_transpose_kernel<T>, grid, dim3(256), 0, st, (const T*)d.w, (char*)wt, d.cout,
                                         d.cin, d.r, d.s, d.stride, gp));
  return hipGetLastError();
}

hipError_t maxpool_forward(const void* x, void* y, int n, int h, int wd, int c, int r, int s,
                           int stride, int pad, int dtype, hipStream_t st) {
  if (!x || !y || n <= 0 || h <= 0 || wd <= 0 || c <= 0 || (c & 3) || r <= 0 || s <= 0 || stride <= 0 ||
      pad < 0 || pad >= r || pad >= s)
    return hipErrorInvalidValue;
  const int ho = (h + 2 * pad - r) / stride + 1, wo = (wd + 2 * pad - s) / stride + 1;
  if (ho <= 0 || wo <= 0) return hipErrorInvalidValue;
  const size_t total = (size_t)n * ho * wo * (c / 4);
  const int v = dtype == DT_BF16 ? 8 : 4;
  const size_t wide = total * 4 / v;
  if (r == 3 && s == 3 && c % v == 0 && wide <= (size_t)1 << 30 && !((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & 15)) {
    const unsigned blocks = grid_for(wide, 256 * 64);
    if (dtype == DT_F32)
      hipLaunchKernelGGL((maxpool3_fwd_kernel<float, 4>), dim3(blocks), dim3(THREADS), 0, st, (const float*)x, (float*)y, (int)wide, h, wd, c, stride, pad, ho, wo);
    else if (dtype == DT_BF16)
      hipLaunchKernelGGL((maxpool3_fwd_kernel<bf16_t, 8>), dim3(blocks), dim3(THREADS), 0, st, (const bf16_t*)x, (bf16_t*)y, (int)wide, h, wd, c, stride, pad, ho, wo);
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  }
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(maxpool_fwd_kernel<T>, dim3(grid_for(total)), dim3(THREADS), 0, st,
                                         (const T*)x, (T*)y, n, h, wd, c, r, s, stride, pad, ho, wo));
  return hipGetLastError();
}

hipError_t maxpool_backward(const void* x, const void* dy, void* dx, int n, int h, int wd, int c,
                            int r, int s, int stride, int pad, int accumulate, int dtype, hipStream_t st) {
  if (!x || !dy || !dx || n <= 0 || h <= 0 || wd <= 0 || c <= 0 || r <= 0 || s <= 0 || stride <= 0 ||
      pad < 0 || pad >= r || pad >= s)
    return hipErrorInvalidValue;
  const int ho = (h + 2 * pad - r) / stride + 1, wo = (wd + 2 * pad - s) / stride + 1;
  if (ho <= 0 || wo <= 0) return hipErrorInvalidValue;
  if (c % 4 == 0 && r == 3 && s == 3 && stride == 2 && pad == 1) {
    const size_t blocks = (size_t)n * ((h + 1) / 2) * ((wd + 1) / 2) * (c / 4);
    const int strip = maxpool_strip(blocks, dt_size(dtype));
    const size_t total = (size_t)n * (((h + 1) / 2 + strip - 1) / strip) * ((wd + 1) / 2) * (c / 4);
    ACC_DISPATCH(dtype, hipLaunchKernelGGL(maxpool3s2_bwd_kernel<T>, dim3(grid_for(total, 256 * 64)), dim3(THREADS), 0, st,
                                           (const T*)x, (const T*)dy, (T*)dx, n, h, wd, c, ho, wo, accumulate, strip));
  } else if (c % 4 == 0) {
    const size_t total = (size_t)n * h * wd * (c / 4);
    ACC_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_bwd_kernel<T, 4>), dim3(grid_for(total, 256 * 64)), dim3(THREADS), 0,
                                           st, (const T*)x, (const T*)dy, (T*)dx, n, h, wd, c, r, s, stride, pad, ho,
                                           wo, accumulate));
  } else {
    const size_t total = (size_t)n * h * wd * c;
    ACC_DISPATCH(dtype, hipLaunchKernelGGL((maxpool_bwd_kernel<T, 1>), dim3(grid_for(total, 256 * 64)), dim3(THREADS), 0,
                                           st, (const T*)x, (const T*)dy, (T*)dx, n, h, wd, c, r, s, stride, pad, ho,
                                           wo, accumulate));
  }
  return hipGetLastError();
}

namespace {
// four channels at a time: whole groups of four, addresses that allow the wide access, grid sizes within bounds
inline bool gap_wide(const void* x, const void* y, int c, int dtype) {
  const uintptr_t mask = dtype == DT_BF16 ? 7 : 15;
  return c % 4 == 0 && !((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & mask) && c / 4 <= 64 * 65535;
}
}  // namespace

hipError_t gap_forward(const void* x, void* y, int n, int hw, int c, int dtype, hipStream_t st) {
  if (!x || !y || n <= 0 || hw <= 0 || c <= 0) return hipErrorInvalidValue;
  if (gap_wide(x, y, c, dtype)) {
    const int tpr = c / 4 < 64 ? c / 4 : 64, rpi = THREADS / tpr, slices = (c / 4 + tpr - 1) / tpr;
    ACC_DISPATCH(dtype, hipLaunchKernelGGL(gap_fwd4_kernel<T>, dim3(n < kGapImages ? n : kGapImages, slices), dim3(THREADS), 0, st, (const T*)x,
                                           (T*)y, n, hw, c, tpr, rpi));
    return hipGetLastError();
  }
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(gap_fwd_kernel<T>, dim3(grid_for((size_t)n * c)), dim3(THREADS), 0, st,
                                         (const T*)x, (T*)y, n, hw, c));
  return hipGetLastError();
}

hipError_t gap_backward(const void* dy, void* dx, int n, int hw, int c, int accumulate, int dtype, hipStream_t st) {
  if (!dy || !dx || n <= 0 || hw <= 0 || c <= 0) return hipErrorInvalidValue;
  if (gap_wide(dy, dx, c, dtype)) {
    const int tpr = c / 4 < 64 ? c / 4 : 64, rpi = THREADS / tpr, slices = (c / 4 + tpr - 1) / tpr;
    // rows in pieces of at least four trips of a workgroup, about 1024 workgroups
    long pieces = 1024 / ((long)n * slices) + 1;
    const long most = ((long)hw + 4 * rpi - 1) / (4 * rpi);
    if (pieces > most) pieces = most;
    const int per = (int)((hw + pieces - 1) / pieces);
    ACC_DISPATCH(dtype, hipLaunchKernelGGL(gap_bwd4_kernel<T>, dim3(n < kGapImages ? n : kGapImages, slices, (hw + per - 1) / per), dim3(THREADS),
                                           0, st, (const T*)dy, (T*)dx, n, hw, c, tpr, rpi, per, accumulate));
    return hipGetLastError();
  }
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(gap_bwd_kernel<T>, dim3(grid_for((size_t)n * hw * c)), dim3(THREADS), 0, st,
                                         (const T*)dy, (T*)dx, n, hw, c, accumulate));
  return hipGetLastError();
}

hipError_t bias_add(void* y, const float* b, long rows, int c, int dtype, hipStream_t st, int relu) {
  if (!y || !b || rows <= 0 || c <= 0) return hipErrorInvalidValue;
  const size_t total = (size_t)rows * c;
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(bias_add_kernel<T>, dim3(grid_for(total)), dim3(THREADS), 0, st, (T*)y, b,
                                         total, c, relu));
  return hipGetLastError();
}

size_t relu_bias_workspace_bytes(int c) { return (size_t)RB_MAX_SLABS * c * sizeof(double); }

hipError_t relu_bias_backward(void* dy, const void* y, float* db, long rows, int c, void* workspace, int dtype,
                              hipStream_t st) {
  if (!dy || !db || !workspace || rows <= 0 || c <= 0 || (c & 3)) return hipErrorInvalidValue;
  // threads along the channels first (four channels each), the rest of the workgroup along rows
  const int cgroups = c / 4;
  const int tpr = cgroups < 64 ? cgroups : 64;
  const int rpi = THREADS / tpr;
  const int col_slices = (cgroups + tpr - 1) / tpr;
  // enough slabs to fill the chip, at least 4 trips of the workgroup per slab
  long slabs = (rows + (long)rpi * 4 - 1) / ((long)rpi * 4);
  const long cap = RB_MAX_SLABS / col_slices > 0 ? RB_MAX_SLABS / col_slices : 1;
  if (slabs > cap) slabs = cap;
  if (slabs < 1) slabs = 1;
  const long rows_per_slab = (rows + slabs - 1) / slabs;
  slabs = (rows + rows_per_slab - 1) / rows_per_slab;
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(relu_bias_bwd_kernel<T>, dim3((unsigned)slabs, col_slices), dim3(THREADS), 0, st,
                                         (T*)dy, (const T*)y, (double*)workspace, rows, c, tpr, rpi, rows_per_slab));
  hipLaunchKernelGGL(slab_sum_kernel, dim3((c + THREADS - 1) / THREADS), dim3(THREADS), 0, st, (const double*)workspace,
                     db, (int)slabs, c);
  return hipGetLastError();
}

hipError_t relu_mask(void* dy, const void* y, size_t count, int dtype, hipStream_t st) {
  if (!dy || !y || count == 0) return hipErrorInvalidValue;
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(relu_mask_kernel<T>, dim3(grid_for(count)), dim3(THREADS), 0, st, (T*)dy,
                                         (const T*)y, count));
  return hipGetLastError();
}

hipError_t column_sum(const void* dy, float* db, long rows, int c, int dtype, hipStream_t st) {
  if (!dy || !db || rows <= 0 || c <= 0) return hipErrorInvalidValue;
  ACC_DISPATCH(dtype, hipLaunchKernelGGL(column_sum_kernel<T>, dim3((c + THREADS - 1) / THREADS), dim3(THREADS), 0, st,
                                         (const T*)dy, db, rows, c));
  return hipGetLastError();
}

hipError_t softmax_ce(const void* z, const int32_t* labels, float* loss_rows, float* loss, void* dz, int n, int classes, int dtype,
                      hipStream_t st) {
  if (!z || !labels || n <= 0 || classes <= 0 || (loss_rows && !loss)) return hipErrorInvalidValue;
#define ACC_SOFTMAX(V) \
  ACC_DISPATCH(dtype, hipLaunchKernelGGL((softmax_ce_kernel<T, V>), dim3(n), dim3(THREADS), 0, st, (const T*)z, labels, loss_rows, (T*)dz, n, classes))
  if (classes <= 4 * THREADS) ACC_SOFTMAX(4);
  else ACC_SOFTMAX(0);
#undef ACC_SOFTMAX
  if (loss_rows) hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(64), 0, st, loss_rows, loss, n);
  return hipGetLastError();
}

hipError_t softmax_ce_forward(const void* z, const int32_t* labels, float* loss_rows, float* loss,
                              int n, int classes, int dtype, hipStream_t st) {
  if (!loss_rows) return hipErrorInvalidValue;
  return softmax_ce(z, labels, loss_rows, loss, nullptr, n, classes, dtype, st);
}

hipError_t softmax_ce_backward(const void* z, const int32_t* labels, void* dz, int n, int classes, int dtype,
                               hipStream_t st) {
  if (!dz) return hipErrorInvalidValue;
  return softmax_ce(z, labels, nullptr, nullptr, dz, n, classes, dtype, st);
}

hipError_t sgd_update(float* w, const float* g, float lr, size_t count, void* w_bf16, hipStream_t st) {
  if (!w || !g) return hipErrorInvalidValue;
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(sgd_kernel, dim3(grid_for(count)), dim3(THREADS), 0, st, w, g, lr, count, (bf16_t*)w_bf16);
  return hipGetLastError();
}

hipError_t fill_zero(float* p, size_t count, hipStream_t st) {
  if (!p) return hipErrorInvalidValue;
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(count)), dim3(THREADS), 0, st, p, count);
  return hipGetLastError();
}

}  // namespace acc
