// Side jobs of the launches whose workgroups have 256 or 512 threads and most of a compute unit's LDS: one or two such
// workgroups run per compute unit, so each takes a large piece with all its loads in flight (as 256-thread pieces, one 32 x 32
// tile or 1024 elements each, the 2304 tiles of a 512->512 3x3 filter took nine rounds of the chip: the 1x1 512->2048
// data gradient that carries them 51.9 us against 31.4 for the same product without).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "parts_sum.h"

namespace acc {

// elements of a weight gradient per workgroup: small gradients come in many parts, and their workgroups take fewer
// elements, one per thread (64->256 1x1, 16384 elements in 128 parts: the launch that carries them 56 us with
// 8192 elements per workgroup of 512 threads, 41 with 512)
__host__ __device__ constexpr int wide_reduce_piece(size_t count, int threads) { return count >= (size_t)8192 * 32 ? threads * 16 : threads; }
__host__ __device__ constexpr int wide_flip(int threads) { return threads / 32; }          // 32 x 32 tiles of a filter per workgroup
template <class T> constexpr int wide_scratch(int threads) { return wide_flip(threads) * 32 * 33 * (int)sizeof(T); }

inline long flip_tiles(int cout, int cin, int r, int s) { return (long)((cin + 31) / 32) * ((cout + 31) / 32) * r * s; }
__host__ __device__ inline long wide_reduce_blocks(size_t count, int threads) {
  const size_t piece = wide_reduce_piece(count, threads);
  return (long)((count + piece - 1) / piece);
}
// workgroups of both jobs
inline long wide_side_blocks(const ReduceJob& j, const FlipJob& f, int threads) {
  return wide_reduce_blocks(j.count, threads) + (f.wt ? (flip_tiles(f.cout, f.cin, f.r, f.s) + wide_flip(threads) - 1) / wide_flip(threads) : 0);
}

// piece `id` of the job
template <int THREADS>
__device__ __forceinline__ void reduce_wide(const ReduceJob& j, int id) {
  constexpr int U = 4;
  const int tid = threadIdx.x;
  if (wide_reduce_piece(j.count, THREADS) == THREADS) {
    const size_t i = (size_t)id * THREADS + tid;
    if (i < j.count) j.dw[i] = sum_parts1(j.part + i, j.count, j.splits);
    return;
  }
  const size_t base = (size_t)id * (THREADS * 16) + (size_t)tid * 4;
  if ((j.count & 3) == 0) {
    size_t at[U];
    bool ok[U];
    float4 sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t i = base + (size_t)u * (THREADS * 4);
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
  for (int u = 0; u < U; ++u) add_parts4(j, base + (size_t)u * (THREADS * 4));
}

// THREADS / 32 tiles of 32 x 32 (co, ci) of a flipped, transposed filter; scratch: wide_scratch<T>(THREADS) bytes of LDS
template <class T, int THREADS>
__device__ __forceinline__ void flip_wide(const FlipJob& f, int id, void* scratch) {
  constexpr int SETS = THREADS / 256, FLIP = wide_flip(THREADS);     // 256 threads per tile, eight tiles each
  const int tid = threadIdx.x, tx = tid & 31, ty = (tid >> 5) & 7, hi = tid >> 8;
  const int bx = (f.cin + 31) / 32, by = (f.cout + 31) / 32, tiles = bx * by * f.r * f.s;
  T (*lds)[32][33] = reinterpret_cast<T (*)[32][33]>(scratch);
  const T* w = static_cast<const T*>(f.w);
  T* wt = static_cast<T*>(f.wt);
  T v[8][4];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int t = id * FLIP + SETS * u + hi, tap = t / (bx * by), rem = t - tap * (bx * by);
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
  for (int u = 0; u < 8; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[SETS * u + hi][ty + 8 * i][tx] = v[u][i];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int t = id * FLIP + SETS * u + hi, tap = t / (bx * by), rem = t - tap * (bx * by);
    const int co0 = (rem / bx) * 32, ci0 = (rem - (rem / bx) * bx) * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ci = ci0 + ty + 8 * i, co = co0 + tx;
      if (t < tiles && ci < f.cin && co < f.cout) wt[((size_t)ci * f.r * f.s + tap) * f.cout + co] = lds[SETS * u + hi][tx][ty + 8 * i];
    }
  }
}

// workgroup `id` of those that do a launch's side jobs; every thread of it is here
template <class T, int THREADS>
__device__ __forceinline__ void wide_side_jobs(const ReduceJob& j, const FlipJob& f, int id, void* scratch) {
  const int sums = (int)wide_reduce_blocks(j.count, THREADS);
  if (id < sums) reduce_wide<THREADS>(j, id);
  else flip_wide<T, THREADS>(f, id - sums, scratch);
}

}  // namespace acc
