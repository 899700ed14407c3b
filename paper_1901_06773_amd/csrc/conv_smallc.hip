// Convolutions with a handful of input channels (the 3-channel first layer of every network), forward pass and weight
// gradient.  The channels are too few for the 16-byte chunks the other kernels move, and the per-element loader they
// fall back to spends its time on index arithmetic.  Here a workgroup keeps the input rows of a few output rows
// of one image in LDS, as fp32, zeros around them: the values that output position q reads through filter row kr are
// then s*c consecutive words at  row(kr) + q*stride*c,  and a matrix operand is eight words per lane from there, split
// into bf16 parts on the way (split3.h; with bf16 storage the values are one part, exactly).
// 512 threads, one workgroup per compute unit, which walks over groups of output rows.
//
// Bound: writing the output / reading dy once (3->64 7x7/2 at 224x224, 32 images: 103 MB, 22 us); the products take 20 us
// at the rate the matrix cores sustain.
#include "kernels.h"
#include "dtype.h"
#include "split3.h"

namespace acc {
namespace {

constexpr int SC_THREADS = 512, SC_WAVES = 8;
constexpr int SC_ROW_WORDS = 21 * 1024;                // LDS words for input rows (84 KB)
constexpr int SC_KPAD = 176;                           // forward: K with every filter row padded to whole groups of eight, at most
constexpr int SC_J = 160;                              // weight gradient: filter columns, at most
template <class T> struct Parts { static constexpr int N = sizeof(T) == 4 ? 3 : 1; };

struct SmallGeom {
  int h, wd, c, p, q, r, s, stride, pad;
  int row_words;                                       // LDS words per input row: (wd + 2 * pad) * c, plus what the last group of eight overhangs, even
  int rows;                                            // output rows per group, at most
  uint32_t row_inv;                                    // i / row_words = (i * row_inv) >> 32 for the words of a group
};

// input rows of the output rows [p0, p0 + n_rows) of image img; waits for nothing, the caller synchronises
template <int U, class T>                              // U words of a thread on their way at once
__device__ __forceinline__ void stage_rows(const T* __restrict__ x, const SmallGeom& sg, int img, int p0, int n_rows, float* lds) {
  const int in_rows = (n_rows - 1) * sg.stride + sg.r, len = sg.wd * sg.c, lead = sg.pad * sg.c;
  const int total = in_rows * sg.row_words, iy0 = p0 * sg.stride - sg.pad;
  // addresses count from the group's first row; a word outside the image reads the nearest row's first value and is dropped
  const T* src = x + ((ptrdiff_t)img * sg.h + iy0) * len;
  const int spare = (min(max(iy0, 0), sg.h - 1) - iy0) * len;
#pragma unroll 1
  for (int i0 = threadIdx.x; i0 < total; i0 += U * SC_THREADS) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * SC_THREADS, row = (int)__umulhi((uint32_t)i, sg.row_inv), at = i - row * sg.row_words - lead, iy = iy0 + row;
      const bool ok = (i < total) & ((unsigned)at < (unsigned)len) & ((unsigned)iy < (unsigned)sg.h);
      const float t = Elem<T>::load(src + (ok ? row * len + at : spare));
      v[u] = ok ? t : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * SC_THREADS < total) lds[i0 + u * SC_THREADS] = v[u];
  }
}

// eight values -> one fragment per part
template <int NP>
__device__ __forceinline__ void to_parts(const float (&v)[8], x3_v4u (&f)[NP]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (NP == 3) {
      uint32_t h, m, l;
      x3_split(v[2 * e], v[2 * e + 1], h, m, l);
      f[0][e] = h; f[1][e] = m; f[2][e] = l;
    } else {
      f[0][e] = x3_pack(v[2 * e], v[2 * e + 1]);
    }
  }
}

// the products of two fragments: six with three parts (small terms first), one with one
template <int NP>
__device__ __forceinline__ void product(const x3_v4u (&a)[NP], const x3_v4u (&b)[NP], x3_v16f& acc) {
  if constexpr (NP == 3) {
    acc = x3_mfma(a[2], b[0], acc);
    acc = x3_mfma(a[0], b[2], acc);
    acc = x3_mfma(a[1], b[1], acc);
    acc = x3_mfma(a[1], b[0], acc);
    acc = x3_mfma(a[0], b[1], acc);
  }
  acc = x3_mfma(a[0], b[0], acc);
}

[[maybe_unused]] __device__ __forceinline__ bool any_nonfinite(const x3_v16f& c) {
  float t = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) t = fmaf(c[v], 0.f, t);
  return __any(t != 0.f);
}

// ---- forward: y[m][n] = sum over (kr, j) of x * w.  K runs over filter rows padded to groups of eight (the padded places
// have zero weights).  The filter's parts for 64 output channels stay in LDS, [part][step][channel][16]; a wave takes one
// block of 32 positions in two output rows at a time (2 x 2 blocks of 32 x 32, one K step = 16 values).
template <class T, bool ACT>
__global__ __launch_bounds__(SC_THREADS, 1) void smallc_fwd_kernel(ConvGeom g, SmallGeom sg, int groups_per_img, int n_groups) {
  [[maybe_unused]] constexpr int NP = Parts<T>::N;
  __shared__ __attribute__((aligned(16))) float rows[SC_ROW_WORDS];
  __shared__ __attribute__((aligned(16))) x3_v4u wf[NP * (SC_KPAD / 8) * 64];
#if defined(__HIP_DEVICE_COMPILE__)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const int n0 = blockIdx.y * 64, jl = sg.s * sg.c, g8 = (jl + 7) >> 3, K = sg.r * jl, n_g8 = sg.r * g8, steps = (n_g8 + 1) >> 1;
  // filter -> parts
  for (int i = tid; i < steps * 2 * 64; i += SC_THREADS) {
    const int n = i & 63, grp = i >> 6, kr = grp / g8, j = (grp - kr * g8) * 8;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool ok = n0 + n < g.n_out && kr < sg.r && j + e < jl;
      const float t = Elem<T>::load(static_cast<const T*>(g.w) + (ok ? (size_t)(n0 + n) * K + kr * jl + j + e : 0));
      v[e] = ok ? t : 0.f;
    }
    x3_v4u f[NP];
    to_parts<NP>(v, f);
#pragma unroll
    for (int p = 0; p < NP; ++p) wf[(p * (SC_KPAD / 8) + grp) * 64 + n] = f[p];
  }
  const int qb = (sg.q + 31) >> 5, sc = sg.stride * sg.c;
  for (int grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
    const int img = grp / groups_per_img, p0 = (grp - img * groups_per_img) * sg.rows;
    const int n_rows = min(sg.rows, sg.p - p0), pairs = (n_rows + 1) >> 1;
    __syncthreads();                                   // the rows of the group before are no longer read
    stage_rows<16>(static_cast<const T*>(g.in), sg, img, p0, n_rows, rows);
    __syncthreads();
    for (int unit = wave; unit < pairs * qb; unit += SC_WAVES) {
      const int pr = (unit / qb) * 2, q0 = (unit % qb) * 32;
      x3_v16f acc[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
      // the lane's position; one that does not exist reads the last one's values and is not stored
      const int q = min(q0 + (lane & 31), sg.q - 1);
      const float* base0 = rows + pr * sg.stride * sg.row_words + q * sc;
      const float* base1 = rows + min(pr + 1, n_rows - 1) * sg.stride * sg.row_words + q * sc;
      int kr = half / g8, part = half - kr * g8;        // the lane's group of eight
      for (int s = 0; s < steps; ++s) {
        const int at = min(kr, sg.r - 1) * sg.row_words + part * 8;
        float v0[8], v1[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) { v0[e] = base0[at + e]; v1[e] = base1[at + e]; }
        x3_v4u a[2][NP], b[2][NP];
        to_parts<NP>(v0, a[0]);
        to_parts<NP>(v1, a[1]);
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int j = 0; j < 2; ++j) b[j][p] = wf[(p * (SC_KPAD / 8) + 2 * s + half) * 64 + 32 * j + (lane & 31)];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) product<NP>(a[i], b[j], acc[i][j]);
        part += 2;
        while (part >= g8) { part -= g8; ++kr; }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (pr + i >= n_rows) continue;
        const size_t row0 = ((size_t)img * sg.p + p0 + pr + i) * sg.q;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int n = n0 + 32 * j + (lane & 31);
          if (any_nonfinite(acc[i][j])) {
            // in fp32, every place of the filter on its own (a value beside the window times a padded zero weight, or a part
            // of a value, may have made the block what it is)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
            const float* rb = i == 0 ? base0 : base1;
            for (int k = 0; k < K; k += 2) {
              const int kk = min(k + half, K - 1), fr = kk / jl, fj = kk - fr * jl;
              float av = rb[fr * sg.row_words + fj];
              float bv = n < g.n_out ? Elem<T>::load(static_cast<const T*>(g.w) + (size_t)n * K + kk) : 0.f;
              if (k + half >= K) av = bv = 0.f;
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc[i][j], 0, 0, 0);
            }
          } else if constexpr (NP == 3) {
            acc[i][j] *= kX3Unscale;
          }
          if (n >= g.n_out) continue;
          const float bias_n = ACT && g.bias ? g.bias[n] : 0.f;
          T* o = static_cast<T*>(g.out) + row0 * g.n_out + n;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int qq = q0 + 8 * (v >> 2) + 4 * half + (v & 3);
            float val = acc[i][j][v];
            if constexpr (ACT) {
              val += bias_n;
              if (g.relu) val = fmaxf(val, 0.f);
            }
            if (qq < sg.q) Elem<T>::store(o + (size_t)qq * g.n_out, val);
          }
        }
      }
    }
  }
#else
  (void)rows; (void)wf;
#endif
}

// The same with the rows in LDS as their parts: a value is split once per group of rows and not in each of the filter places that read it
// (twelve of them for 7x7/2), which kept the vector units as busy as the matrix cores.  A fragment is then four words per part
// (five, shifted by half a word, where positions lie an odd number of values apart).  The next group's values are asked for
// before this one's products.  LDS holds two thirds of the rows that words would take; images too wide for one pair of them stay with the kernel above.
// 3->64 7x7/2 at 224x224: fp32, 32 images 77 -> 60 us (128: 263 -> 213); bf16, 128 images 142 -> 101; 448x448, fp32, 8 images
// 101 -> 64; 3x3 of 32 images at 224x224, bf16 87 -> 56. Results leave through a descriptor of their row, an address each and no test.
// In fp32 a second set of fragments, read ahead, does not fit beside the next group's values (spills: 80 us).
// A barrier for what lies in LDS: stores of results stay on their way.
__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);                  // LDS accesses done, any number of vector memory accesses on their way
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#endif
}
template <class T> constexpr int kPairs = Parts<T>::N == 3 ? 7936 : 10752;       // pairs of values in LDS per part
template <class T, bool ACT, bool ODD>
__global__ __launch_bounds__(SC_THREADS, 1) void smallc_fwd_parts_kernel(ConvGeom g, SmallGeom sg, int groups_per_img, int n_groups) {
  [[maybe_unused]] constexpr int NP = Parts<T>::N, PAIRS = kPairs<T>, U = (PAIRS + SC_THREADS - 1) / SC_THREADS;
  __shared__ __attribute__((aligned(16))) uint32_t rows[NP * PAIRS + 4];
  __shared__ __attribute__((aligned(16))) x3_v4u wf[NP * (SC_KPAD / 8) * 64];
#if defined(__HIP_DEVICE_COMPILE__)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const int n0 = blockIdx.y * 64, jl = sg.s * sg.c, g8 = (jl + 7) >> 3, K = sg.r * jl, n_g8 = sg.r * g8, steps = (n_g8 + 1) >> 1;
  const T* const x = static_cast<const T*>(g.in);
  const int len = sg.wd * sg.c, lead = sg.pad * sg.c;
  float nv[2 * U];                                     // the thread's pairs of the next group
  auto ask = [&](int grp) {
    const int img = grp / groups_per_img, p0 = (grp - img * groups_per_img) * sg.rows;
    const int n_rows = min(sg.rows, sg.p - p0), in_rows = (n_rows - 1) * sg.stride + sg.r, total = in_rows * sg.row_words, iy0 = p0 * sg.stride - sg.pad;
    int t = tid;
    asm volatile("" : "+v"(t));                        // places are worked out again for every group: kept, they take 32 registers
    // one image; what lies outside reads as zero
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(x) + (size_t)img * sg.h * len, 0, sg.h * len * (int)sizeof(T), 0x00020000);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = 2 * (t + u * SC_THREADS), row = (int)__umulhi((uint32_t)i, sg.row_inv), at = i - row * sg.row_words - lead, iy = iy0 + row;
      const bool in = (i < total) & ((unsigned)iy < (unsigned)sg.h);   // (row_words is even: a pair lies in one row)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int off = in & ((unsigned)(at + e) < (unsigned)len) ? (iy * len + at + e) * (int)sizeof(T) : (int)0x7ffffff0;
        if constexpr (NP == 3) nv[2 * u + e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
        else nv[2 * u + e] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0));   // the bf16 itself
      }
    }
  };
  auto put = [&]() {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = tid + u * SC_THREADS;
      if (i >= PAIRS) continue;
      if constexpr (NP == 3) {
        uint32_t h, m, l;
        x3_split(nv[2 * u], nv[2 * u + 1], h, m, l);
        rows[i] = h; rows[PAIRS + i] = m; rows[2 * PAIRS + i] = l;
      } else {
        rows[i] = __float_as_uint(nv[2 * u]) | __float_as_uint(nv[2 * u + 1]) << 16;
      }
    }
  };
  if ((int)blockIdx.x < n_groups) ask(blockIdx.x);
  // filter -> parts
  for (int i = tid; i < steps * 2 * 64; i += SC_THREADS) {
    const int n = i & 63, grp = i >> 6, kr = grp / g8, j = (grp - kr * g8) * 8;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool ok = n0 + n < g.n_out && kr < sg.r && j + e < jl;
      const float t = Elem<T>::load(static_cast<const T*>(g.w) + (ok ? (size_t)(n0 + n) * K + kr * jl + j + e : 0));
      v[e] = ok ? t : 0.f;
    }
    x3_v4u f[NP];
    to_parts<NP>(v, f);
#pragma unroll
    for (int p = 0; p < NP; ++p) wf[(p * (SC_KPAD / 8) + grp) * 64 + n] = f[p];
  }
  const int qb = (sg.q + 31) >> 5, sc = sg.stride * sg.c;
  for (int grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
    const int img = grp / groups_per_img, p0 = (grp - img * groups_per_img) * sg.rows;
    const int n_rows = min(sg.rows, sg.p - p0), pairs = (n_rows + 1) >> 1;
    lds_barrier();                                     // the rows of the group before are no longer read
    put();
    lds_barrier();
    if (grp + (int)gridDim.x < n_groups) ask(grp + gridDim.x);
    for (int unit = wave; unit < pairs * qb; unit += SC_WAVES) {
      const int pr = (unit / qb) * 2, q0 = (unit % qb) * 32;
      x3_v16f acc[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
      // the lane's position; one that does not exist reads the last one's values and is not stored
      const int q = min(q0 + (lane & 31), sg.q - 1);
      const int base0 = pr * sg.stride * sg.row_words + q * sc, base1 = min(pr + 1, n_rows - 1) * sg.stride * sg.row_words + q * sc;
      const uint32_t odd = ODD ? (uint32_t)(q * sc & 1) * 16u : 0u;     // bits
      struct Frags { x3_v4u a[2][NP], b[2][NP]; };
      int kr = half / g8, part = half - kr * g8;        // the lane's group of eight
      auto read = [&](Frags& f, int s) {
        const int at = min(kr, sg.r - 1) * sg.row_words + part * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            const uint32_t* w = rows + p * PAIRS + (((i == 0 ? base0 : base1) + at) >> 1);
            if constexpr (ODD) {
              const uint32_t t[5] = {w[0], w[1], w[2], w[3], w[4]};
#pragma unroll
              for (int e = 0; e < 4; ++e) f.a[i][p][e] = __builtin_amdgcn_alignbit(t[e + 1], t[e], odd);
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) f.a[i][p][e] = w[e];
            }
          }
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int j = 0; j < 2; ++j) f.b[j][p] = wf[(p * (SC_KPAD / 8) + 2 * s + half) * 64 + 32 * j + (lane & 31)];
        part += 2;
        while (part >= g8) { part -= g8; ++kr; }
      };
      auto multiply = [&](const Frags& f) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) product<NP>(f.a[i], f.b[j], acc[i][j]);
      };
      if constexpr (NP == 3) {
#pragma unroll 1
        for (int s = 0; s < steps; ++s) {
          Frags f;
          read(f, s);
          multiply(f);
        }
      } else {
      Frags f0, f1;
      read(f0, 0);
#pragma unroll 1
      for (int s = 0; s < steps; s += 2) {
        if (s + 1 < steps) read(f1, s + 1);
        __builtin_amdgcn_sched_barrier(0);             // (a third set of fragments does not fit)
        multiply(f0);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 >= steps) break;
        if (s + 2 < steps) read(f0, s + 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f1);
        __builtin_amdgcn_sched_barrier(0);
      }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (pr + i >= n_rows) continue;
        // one row of results; positions and channels that do not exist are stored outside of it, which drops them
        const size_t row0 = ((size_t)img * sg.p + p0 + pr + i) * sg.q;
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(static_cast<T*>(g.out) + row0 * g.n_out, 0, sg.q * g.n_out * (int)sizeof(T), 0x00020000);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int n = n0 + 32 * j + (lane & 31);
          if (any_nonfinite(acc[i][j])) {
            // in fp32, from memory (a value beside the window times a padded zero weight, or a part of a value, may have
            // made the block what it is)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
            for (int k = 0; k < K; k += 2) {
              const int kk = min(k + half, K - 1), fr = kk / jl, fj = kk - fr * jl;
              const int iy = (p0 + pr + i) * sg.stride - sg.pad + fr, at = q * sc - lead + fj;
              const bool in = k + half < K && (unsigned)iy < (unsigned)sg.h && (unsigned)at < (unsigned)len;
              float av = in ? Elem<T>::load(x + ((size_t)img * sg.h + iy) * len + at) : 0.f;
              float bv = k + half < K && n < g.n_out ? Elem<T>::load(static_cast<const T*>(g.w) + (size_t)n * K + kk) : 0.f;
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc[i][j], 0, 0, 0);
            }
          } else if constexpr (NP == 3) {
            acc[i][j] *= kX3Unscale;
          }
          const float bias_n = ACT && g.bias ? g.bias[min(n, g.n_out - 1)] : 0.f;
          const int at = n < g.n_out ? ((q0 + 4 * half) * g.n_out + n) * (int)sizeof(T) : (int)0x7f000000;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float val = acc[i][j][v];
            if constexpr (ACT) {
              val += bias_n;
              if (g.relu) val = fmaxf(val, 0.f);
            }
            const int off = at + (8 * (v >> 2) + (v & 3)) * g.n_out * (int)sizeof(T);
            if constexpr (NP == 3) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val), ro, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b16((uint16_t)x3_pack(val, val), ro, off, 0, 0);
          }
        }
      }
    }
  }
#else
  (void)rows; (void)wf;
#endif
}

// Input rows as stage_rows() places them, from global memory straight into LDS: 64 consecutive words per instruction; bf16 values arrive as the
// low halves of their words.  What lies outside the image reads as zero.  The caller waits for the loads.
template <class T>
__device__ __forceinline__ void stage_rows_direct(const T* __restrict__ x, const SmallGeom& sg, int img, int p0, int n_rows, float* lds, int wave, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef __attribute__((address_space(3))) void* lds_ptr;
  const int in_rows = (n_rows - 1) * sg.stride + sg.r, len = sg.wd * sg.c, lead = sg.pad * sg.c;
  const int total = in_rows * sg.row_words, iy0 = p0 * sg.stride - sg.pad;
  const int lo = min(max(iy0, 0), sg.h), hi = max(min(iy0 + in_rows, sg.h), lo);             // rows of the image among them
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(x) + ((size_t)img * sg.h + lo) * len, 0, (hi - lo) * len * (int)sizeof(T), 0x00020000);
  const uint32_t to = (uint32_t)(size_t)lds;
#pragma unroll 4
  for (int i0 = wave * 64; i0 < total; i0 += SC_THREADS) {
    const int i = i0 + lane, row = (int)__umulhi((uint32_t)i, sg.row_inv), at = i - row * sg.row_words - lead, iy = iy0 + row;
    const bool ok = (i < total) & ((unsigned)at < (unsigned)len) & ((unsigned)iy < (unsigned)sg.h);
    const int off = ok ? ((iy - lo) * len + at) * (int)sizeof(T) : (int)0x7ffffff0;
    if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(size_t)(to + i0 * 4), 4, off, 0, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(size_t)(to + i0 * 4), 2, off, 0, 0, 0);
  }
#endif
}
static_assert(SC_ROW_WORDS % 64 == 0, "an instruction writes 64 words");

// ---- weight gradient: dw[co][j] = sum_m dy[m][co] * X[m][j], j = (kr, kt, ci) <= 160 columns, 64 output channels per
// workgroup column.  A step is 16 positions of one output row: dy comes straight from memory (eight positions per lane), X
// from the rows in LDS, every lane at its own columns' places.  The waves take every eighth step of a group of rows and keep
// the whole 64 x 160 block (2 x 5 blocks of 32 x 32); the workgroup adds them up at the end and writes one part.
// Bound by vector instructions beside the matrix cores, and by trips to memory (the sums take 160 registers, so few loads can be on their
// way): the rows go into LDS without passing through registers, all of a group's words at once, and the dy values of the next step
// are asked for a step ahead, through a descriptor that gives zeros outside (a test on the value waits for it where it is asked for).
// With the sum of the parts, 3->64 7x7/2 at 224x224, fp32, 32 images 110 -> 76 us (rows alone 102); bf16, 128 images 254 -> 114
// (rows alone 227); 3x3, bf16, 32 images 231 -> 97.
template <class T>
__global__ __launch_bounds__(SC_THREADS, 1) void smallc_wgrad_kernel(WgradGeom g, SmallGeom sg, int rows_total, int rows_per_split,
                                                                      float* out, size_t split_stride) {
  [[maybe_unused]] constexpr int NP = Parts<T>::N, NJ = SC_J / 32;
  __shared__ __attribute__((aligned(16))) float rows[SC_ROW_WORDS];
#if defined(__HIP_DEVICE_COMPILE__)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const int co0 = blockIdx.y * 64, jl = sg.s * sg.c, J = sg.r * jl, sc = sg.stride * sg.c;
  const int lo = blockIdx.x * rows_per_split, hi = min(lo + rows_per_split, rows_total);   // output rows of the minibatch
  int col[NJ];                                         // LDS place of the lane's columns at position 0
#pragma unroll
  for (int b = 0; b < NJ; ++b) {
    const int j = min(32 * b + (lane & 31), J - 1), kr = j / jl;
    col[b] = kr * sg.row_words + j - kr * jl;
  }
  x3_v16f acc[2][NJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int b = 0; b < NJ; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][b][v] = 0.f;
  const int spr = (sg.q + 15) >> 4;                    // steps per output row
  auto fragment = [](const float (&v)[8], x3_v4u (&f)[NP]) {
    if constexpr (NP == 3) {
      to_parts<NP>(v, f);
    } else {                                           // a bf16 in the low half of each word
#pragma unroll
      for (int e = 0; e < 4; ++e) f[0][e] = __float_as_uint(v[2 * e]) | __float_as_uint(v[2 * e + 1]) << 16;
    }
  };
  const T* dy = static_cast<const T*>(g.dy);
  const bool c_ok[2] = {co0 + (lane & 31) < g.cout, co0 + 32 + (lane & 31) < g.cout};
  for (int r0 = lo; r0 < hi;) {
    const int img = r0 / sg.p, p0 = r0 - img * sg.p, n_rows = min(min(sg.rows, sg.p - p0), hi - r0);
    // positions and channels that do not exist read as zero (without a test on the value, which would wait for it here)
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(dy) + (size_t)r0 * sg.q * g.cout, 0,
                                                                        n_rows * sg.q * g.cout * (int)sizeof(T), 0x00020000);
    auto load = [&](int s, float (&v)[2][8]) {
      const int row = s / spr, q = (s - row * spr) * 16 + half * 8;
      const int at = ((row * sg.q + q) * g.cout + co0 + (lane & 31)) * (int)sizeof(T);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int off = c_ok[i] & (q + e < sg.q) ? at + (e * g.cout + 32 * i) * (int)sizeof(T) : (int)0x7ffffff0;
          if constexpr (NP == 3) v[i][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rd, off, 0, 0));
          else v[i][e] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rd, off, 0, 0));   // the bf16 itself
        }
    };
    const int n_steps = n_rows * spr;
    float nv[2][8];
    if (wave < n_steps) load(wave, nv);                // on its way while the rows are staged
    __syncthreads();
    stage_rows_direct(static_cast<const T*>(g.x), sg, img, p0, n_rows, rows, wave, lane);
    __builtin_amdgcn_s_waitcnt(0x0070);                // this wave's loads have landed, in LDS too
    __syncthreads();
    for (int s = wave; s < n_steps; s += SC_WAVES) {
      x3_v4u a[2][NP];
      fragment(nv[0], a[0]);
      fragment(nv[1], a[1]);
      if (s + SC_WAVES < n_steps) load(s + SC_WAVES, nv);
      const int row = s / spr, q = (s - row * spr) * 16 + half * 8;
      const float* base = rows + row * sg.stride * sg.row_words;
      int at[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) at[e] = min(q + e, sg.q - 1) * sc;   // a position that does not exist meets dy = 0
#pragma unroll
      for (int b = 0; b < NJ; ++b) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = base[col[b] + at[e]];
        x3_v4u f[NP];
        fragment(v, f);
        product<NP>(a[0], f, acc[0][b]);
        product<NP>(a[1], f, acc[1][b]);
      }
    }
    r0 += n_rows;
  }
  // the waves' sums, a column block at a time: [wave][co][32] through LDS, added in wave order
  float* dst = out + (size_t)blockIdx.x * split_stride;
#pragma unroll
  for (int b = 0; b < NJ; ++b) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        rows[(wave * 64 + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3)) * 32 + (lane & 31)] = acc[i][b][v];
    __syncthreads();
    for (int e = tid; e < 64 * 32; e += SC_THREADS) {
      const int co = e >> 5, j = 32 * b + (e & 31);
      float sum = rows[e];
#pragma unroll
      for (int w = 1; w < SC_WAVES; ++w) sum += rows[w * 64 * 32 + e];
      if (co0 + co >= g.cout || j >= J) continue;
      if (!(fabsf(sum) <= 3.402823466e38f)) {
        // not finite: this element in fp32 (a part of a value, or a value beside the row times a zero, may have done it)
        const int kr = j / jl, off = j - kr * jl, kt = off / sg.c, ci = off - kt * sg.c;
        float t = 0.f;
        for (int rr = lo; rr < hi; ++rr) {
          const int im = rr / sg.p, iy = (rr - im * sg.p) * sg.stride + kr - sg.pad;
          for (int q = 0; q < sg.q; ++q) {
            const int ix = q * sg.stride + kt - sg.pad;
            const bool in = (unsigned)iy < (unsigned)sg.h && (unsigned)ix < (unsigned)sg.wd;
            const float xv = in ? Elem<T>::load(static_cast<const T*>(g.x) + (((size_t)im * sg.h + iy) * sg.wd + ix) * sg.c + ci) : 0.f;
            t = fmaf(Elem<T>::load(dy + ((size_t)rr * sg.q + q) * g.cout + co0 + co), xv, t);
          }
        }
        sum = t;
      } else if constexpr (NP == 3) {
        sum *= kX3Unscale;
      }
      dst[(size_t)(co0 + co) * J + j] = sum;
    }
  }
#else
  (void)rows;
#endif
}

static_assert(SC_WAVES * 64 * 32 <= SC_ROW_WORDS, "the waves' sums");

// Rows per group (0: the shape is not taken): as many as their input rows fit in LDS, at most eight
SmallGeom small_geom(int h, int wd, int c, int p, int q, int r, int s, int stride, int pad) {
  SmallGeom sg{h, wd, c, p, q, r, s, stride, pad, 0, 0, 0};
  const long words = (long)(wd + 2 * pad) * c + 8;
  if (words > SC_ROW_WORDS) return sg;
  sg.row_words = (int)((words + 1) & ~1L);
  sg.row_inv = (uint32_t)(((1ull << 32) + sg.row_words - 1) / sg.row_words);   // exact while i * row_words < 2^32
  for (int n = 8; n >= 1; --n)
    if ((long)((n - 1) * stride + r) * sg.row_words <= SC_ROW_WORDS) { sg.rows = n < p ? n : p; break; }
  return sg;
}

}  // namespace

// Few channels, a filter whose padded rows fit the LDS image, a plain dense result, and enough groups of output rows: a workgroup
// takes one at a time (times 64 output channels), and with few of them the per-element kernel's many small workgroups
// finish first.  Where the line lies, workgroups: per-element -> this kernel.  fp32: 7x7/2 at 224x224 84: 31 -> 38 us,
// 112: 41 -> 39, 224: 69 -> 41; 3x3 at 224x224 112: 27 -> 29, 168: 37 -> 30; 3->128 at 128x128 128: 19 -> 19, 256: 33 -> 21.
// bf16: 7x7/2 42: 21 -> 22, 56: 24 -> 23, 84: 31 -> 23; 3x3 28: 15 -> 23, 56: 25 -> 24, 84: 33 -> 24; 3->128 64: 16 -> 16, 128: 27 -> 17.
// And enough units of two rows by 32 columns in a group for its eight waves (32x32 maps have four: fp32 3->64 3x3, 256 images
// 31 -> 33); in fp32, filters that read values more than once (4x4/4 at 224x224, 48 images 29 -> 31).
bool conv_smallc_takes(const ConvGeom& g, long M) {
  if (g.c > 4 || g.c % 4 == 0 || g.r * ((g.s * g.c + 7) / 8) * 8 > SC_KPAD - 8 || g.stats || g.bnb.sums || g.accumulate || g.side.count || g.flip.wt ||
      g.out_stride != 1 || g.out_h != g.p || g.out_w != g.q || g.pad_dx != 0 || M < 16384 || (g.dtype == DT_F32 && g.stride >= g.r))
    return false;
  // every place the rows in LDS are read at lies inside the padded input: (q-1)*stride + s <= wd + 2*pad, likewise rows
  if ((g.q - 1) * (long)g.stride + g.s > g.wd + 2L * g.pad || (g.p - 1) * (long)g.stride + g.r > g.h + 2L * g.pad) return false;
  const SmallGeom sg = small_geom(g.h, g.wd, g.c, g.p, g.q, g.r, g.s, g.stride, g.pad);
  const long cols = (g.n_out + 63) / 64;
  if (sg.rows < 1 || cols > 65535) return false;
  const long groups = (long)g.n_img * ((g.p + sg.rows - 1) / sg.rows), units = (sg.rows + 1) / 2 * ((g.q + 31L) / 32);
  return units >= SC_WAVES && (groups < 256 ? groups : 256) * cols >= (g.dtype == DT_F32 ? 144 : 72);
}

hipError_t conv_smallc_fwd(const ConvGeom& g, hipStream_t st, LaunchProbe* probe) {
  SmallGeom sg = small_geom(g.h, g.wd, g.c, g.p, g.q, g.r, g.s, g.stride, g.pad);
  // rows held as parts: as many as fit, in pairs; one pair at least
  const long room = g.dtype == DT_F32 ? 2 * kPairs<float> : 2 * kPairs<bf16_t>;
  auto values = [&](int rows) { return (long)((rows - 1) * sg.stride + sg.r) * sg.row_words; };
  int rows = sg.rows;
  while (rows > 2 && values(rows) > room) rows = (rows - 1) & ~1;
  const bool parts = rows > 0 && values(rows) <= room && (long)sg.h * sg.wd * sg.c < (1L << 28) && (long)(sg.q + 32) * g.n_out < (1L << 28);
  if (parts) sg.rows = rows;
  const int per_img = sg.rows < 1 ? 0 : (g.p + sg.rows - 1) / sg.rows;
  const long groups = (long)per_img * g.n_img;
  if (sg.rows < 1 || groups > (1L << 30)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(groups < 256 ? groups : 256), (g.n_out + 63) / 64);
  probe->variant = V_SMALLC_FWD;
  probe->kernel = "smallc";
  if (probe->dry) return hipSuccess;
  if (probe->before) (void)hipEventRecord(probe->before, st);
  const bool act = g.bias || g.relu, odd = (sg.stride * sg.c & 1) != 0;
#define ACC_SC(T, A) do { \
    if (!parts) hipLaunchKernelGGL((smallc_fwd_kernel<T, A>), grid, dim3(SC_THREADS), 0, st, g, sg, per_img, (int)groups); \
    else if (odd) hipLaunchKernelGGL((smallc_fwd_parts_kernel<T, A, true>), grid, dim3(SC_THREADS), 0, st, g, sg, per_img, (int)groups); \
    else hipLaunchKernelGGL((smallc_fwd_parts_kernel<T, A, false>), grid, dim3(SC_THREADS), 0, st, g, sg, per_img, (int)groups); } while (0)
  if (g.dtype == DT_F32) { if (act) ACC_SC(float, true); else ACC_SC(float, false); }
  else { if (act) ACC_SC(bf16_t, true); else ACC_SC(bf16_t, false); }
#undef ACC_SC
  if (probe->after) (void)hipEventRecord(probe->after, st);
  return hipGetLastError();
}

// In fp32 the six products of all 160 columns are made however few of them exist, and the per-element kernel is the faster one for
// short filter rows and for few positions: 3x3 of 3 channels at 224x224, 4 / 16 / 32 / 64 images 71 / 155 / 267 / 488 us there,
// 63 / 142 / 317 / 613 here; 7x7/2, 4 (50 thousand positions) / 6 / 8 (100 thousand) / 32 images 49 / 57 / 67 / 189, 49 / 57 / 63 / 94.
int wgrad_smallc_splits(long Mrows, int cin, int cout, int r, int s, int dtype) {
  if (cin > 4 || cin % 4 == 0 || r * s * cin > SC_J || Mrows < 16384) return 0;
  if (dtype == DT_F32 && (r * s * cin <= 96 || Mrows < 80000)) return 0;
  const long want = Mrows / 1024;
  return (int)(want < 256 ? want : 256);
}

bool conv_wgrad_smallc_takes(const WgradGeom& g) {
  const long M = (long)g.n_img * g.p * g.q;
  if (!wgrad_smallc_splits(M, g.cin, g.cout, g.r, g.s, g.dtype) || g.side.count || g.flip_wt || (g.cout + 63) / 64 > 65535 ||
      (g.q + 32L) * g.cout >= (1L << 25))
    return false;
  if ((g.q - 1) * (long)g.stride + g.s > g.wd + 2L * g.pad || (g.p - 1) * (long)g.stride + g.r > g.h + 2L * g.pad) return false;
  return small_geom(g.h, g.wd, g.cin, g.p, g.q, g.r, g.s, g.stride, g.pad).rows > 0;
}

// out: `splits` parts of cout * r*s*cin elements (or dw itself if one)
hipError_t conv_wgrad_smallc(const WgradGeom& g, int splits, float* out, size_t count, hipStream_t st) {
  const SmallGeom sg = small_geom(g.h, g.wd, g.cin, g.p, g.q, g.r, g.s, g.stride, g.pad);
  const int total = g.n_img * g.p, per = (total + splits - 1) / splits;
  const dim3 grid(splits, (g.cout + 63) / 64);
  if (g.dtype == DT_F32)
    hipLaunchKernelGGL(smallc_wgrad_kernel<float>, grid, dim3(SC_THREADS), 0, st, g, sg, total, per, out, count);
  else
    hipLaunchKernelGGL(smallc_wgrad_kernel<bf16_t>, grid, dim3(SC_THREADS), 0, st, g, sg, total, per, out, count);
  return hipGetLastError();
}

}  // namespace acc
