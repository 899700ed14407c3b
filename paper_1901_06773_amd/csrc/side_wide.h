// Side jobs of the launches whose workgroups have 512 threads and most of a compute unit's LDS: one such workgroup
// runs per compute unit, so each takes a large piece with all its loads in flight (as 256-thread pieces, one 32 x 32
// tile or 1024 elements each, the 2304 tiles of a 512->512 3x3 filter took nine rounds of the chip: the 1x1 512->2048
// data gradient that carries them 51.9 us against 31.4 for the same product without).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "parts_sum.h"

namespace acc {

// elements of a weight gradient per workgroup: small gradients come in many parts, and their workgroups take fewer
// elements, one per thread (64->256 1x1, 16384 elements in 128 parts: the launch that carries them 56 us with
// 8192 elements per workgroup, 41 with 512)
__host__ __device__ inline int wide_reduce_piece(size_t count) { return count >= (size_t)8192 * 32 ? 8192 : 512; }
constexpr int kWideFlip = 16;          // 32 x 32 tiles of a filter per workgroup
constexpr int kWideScratch = kWideFlip * 32 * 33 * 4;

inline long flip_tiles(int cout, int cin, int r, int s) { return (long)((cin + 31) / 32) * ((cout + 31) / 32) * r * s; }
__host__ __device__ inline long wide_reduce_blocks(size_t count) {
  const size_t piece = wide_reduce_piece(count);
  return (long)((count + piece - 1) / piece);
}
inline long wide_flip_blocks(int cout, int cin, int r, int s) { return (flip_tiles(cout, cin, r, s) + kWideFlip - 1) / kWideFlip; }

// piece `id` of the job
__device__ __forceinline__ void reduce_wide(const ReduceJob& j, int id) {
  constexpr int U = 4;
  const int tid = threadIdx.x;
  if (wide_reduce_piece(j.count) == 512) {
    const size_t i = (size_t)id * 512 + tid;
    if (i < j.count) j.dw[i] = sum_parts1(j.part + i, j.count, j.splits);
    return;
  }
  const size_t base = (size_t)id * 8192 + (size_t)tid * 4;
  if ((j.count & 3) == 0) {
    size_t at[U];
    bool ok[U];
    float4 sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = base + (size_t)u * 2048;
      ok[u] = i < j.count;
      at[u] = ok[u] ? i : 0;
      sum[u] = *reinterpret_cast<const float4*>(j.part + at[u]);
    }
    int k = 1;
    for (; k + 4 <= j.splits; k += 4) {
      float4 v[4][U];
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int u = 0; u < U; ++u) v[p][u] = *reinterpret_cast<const float4*>(j.part + (size_t)(k + p) * j.count + at[u]);
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int u = 0; u < U; ++u) { sum[u].x += v[p][u].x; sum[u].y += v[p][u].y; sum[u].z += v[p][u].z; sum[u].w += v[p][u].w; }
    }
    for (; k < j.splits; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float4 v = *reinterpret_cast<const float4*>(j.part + (size_t)k * j.count + at[u]);
        sum[u].x += v.x; sum[u].y += v.y; sum[u].z += v.z; sum[u].w += v.w;
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (ok[u]) *reinterpret_cast<float4*>(j.dw + at[u]) = sum[u];
    return;
  }
  for (int u = 0; u < U; ++u) add_parts4(j, base + (size_t)u * 2048);
}

// sixteen 32 x 32 (co, ci) tiles of a flipped, transposed fp32 filter; scratch: kWideScratch bytes of LDS
__device__ __forceinline__ void flip_wide(const FlipJob& f, int id, void* scratch) {
  const int tid = threadIdx.x, tx = tid & 31, ty = (tid >> 5) & 7, hi = tid >> 8;
  const int bx = (f.cin + 31) / 32, by = (f.cout + 31) / 32, tiles = bx * by * f.r * f.s;
  float (*lds)[32][33] = reinterpret_cast<float (*)[32][33]>(scratch);
  const float* w = static_cast<const float*>(f.w);
  float* wt = static_cast<float*>(f.wt);
  float v[kWideFlip / 2][4];
#pragma unroll
  for (int u = 0; u < kWideFlip / 2; ++u) {
    const int t = id * kWideFlip + 2 * u + hi, tap = t / (bx * by), rem = t - tap * (bx * by);
    const int co0 = (rem / bx) * 32, ci0 = (rem - (rem / bx) * bx) * 32;
    const int src = (f.r - 1 - tap / f.s) * f.s + (f.s - 1 - tap % f.s);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int co = co0 + ty + 8 * i, ci = ci0 + tx;
      const bool ok = t < tiles && co < f.cout && ci < f.cin;
      v[u][i] = w[ok ? ((size_t)co * f.r * f.s + src) * f.cin + ci : 0];
    }
  }
#pragma unroll
  for (int u = 0; u < kWideFlip / 2; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[2 * u + hi][ty + 8 * i][tx] = v[u][i];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kWideFlip / 2; ++u) {
    const int t = id * kWideFlip + 2 * u + hi, tap = t / (bx * by), rem = t - tap * (bx * by);
    const int co0 = (rem / bx) * 32, ci0 = (rem - (rem / bx) * bx) * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ci = ci0 + ty + 8 * i, co = co0 + tx;
      if (t < tiles && ci < f.cin && co < f.cout) wt[((size_t)ci * f.r * f.s + tap) * f.cout + co] = lds[2 * u + hi][tx][ty + 8 * i];
    }
  }
}

}  // namespace acc
