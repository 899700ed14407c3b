// Adding up the parts of a weight gradient: dw[i] = part[0][i] + part[1][i] + ..., in that order wherever it is done (a launch of
// its own, or extra workgroups of another one), so that a gradient has the same bits on every way it is computed.
// Several parts are fetched at a time: with hundreds of them (few tiles, many cuts of the minibatch range) one load
// waiting for the sum before it is a chain of latencies.  The parts that fill no batch are fetched together too, with bounds that the
// whole batches do without.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace acc {

// one element: the sum of p[0], p[count], p[2 * count], ...
__device__ __forceinline__ float sum_parts1(const float* p, size_t count, int splits) {
  constexpr int U = 32;
  float sum = p[0];
  int k = 1;
  for (; k + U <= splits; k += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[(size_t)(k + u) * count];
#pragma unroll
    for (int u = 0; u < U; ++u) sum += v[u];
  }
  if (k < splits) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[k + u < splits ? (size_t)(k + u) * count : 0];   // beyond the last part: read, not added
#pragma unroll
    for (int u = 0; u < U; ++u) sum = k + u < splits ? sum + v[u] : sum;
  }
  return sum;
}

// the elements i4 .. i4 + 3 (as far as they exist)
__device__ __forceinline__ void add_parts4(const ReduceJob& j, size_t i4) {
  if (i4 >= j.count) return;
  if ((j.count & 3) == 0) {
    constexpr int U = 8;
    const float* p = j.part + i4;
    float4 sum = *reinterpret_cast<const float4*>(p);
    int k = 1;
    for (; k + U <= j.splits; k += U) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4*>(p + (size_t)(k + u) * j.count);
#pragma unroll
      for (int u = 0; u < U; ++u) { sum.x += v[u].x; sum.y += v[u].y; sum.z += v[u].z; sum.w += v[u].w; }
    }
    if (k < j.splits) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4*>(p + (k + u < j.splits ? (size_t)(k + u) * j.count : 0));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ok = k + u < j.splits;
        sum.x = ok ? sum.x + v[u].x : sum.x;
        sum.y = ok ? sum.y + v[u].y : sum.y;
        sum.z = ok ? sum.z + v[u].z : sum.z;
        sum.w = ok ? sum.w + v[u].w : sum.w;
      }
    }
    *reinterpret_cast<float4*>(j.dw + i4) = sum;
  } else {
    for (size_t i = i4; i < j.count && i < i4 + 4; ++i) j.dw[i] = sum_parts1(j.part + i, j.count, j.splits);
  }
}

}  // namespace acc
