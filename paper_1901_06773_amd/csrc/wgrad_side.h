// Side jobs of a weight-gradient launch: workgroups appended behind the tiles that do small, independent work
// which would otherwise cost a launch of its own.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "parts_sum.h"

namespace acc {

// id: index of the workgroup among the side-job workgroups.  First the
// blocks that add up 1024 elements each of an earlier weight gradient's parts, in their fixed
// order; then the blocks that write one 32 x 32 (co, ci) block each of one tap of the flipped,
// transposed filter.  scratch: at least 32 x 33 elements of LDS.
template <class T>
__device__ __forceinline__ void wgrad_side_jobs(const WgradGeom& g, int id, float* scratch) {
  const ReduceJob& rj = g.side;
  const int reduce_blocks = (int)((rj.count + 1023) / 1024);
  if (id < reduce_blocks) {
    add_parts4(rj, ((size_t)id * 256 + threadIdx.x) * 4);
    return;
  }
  id -= reduce_blocks;
  if (!g.flip_wt) return;
  const int bx = (g.cin + 31) / 32, by = (g.cout + 31) / 32;
  const int tap = id / (bx * by), rem = id - tap * (bx * by);
  const int co0f = (rem / bx) * 32, ci0f = (rem - (rem / bx) * bx) * 32;
  const int kr = g.r - 1 - tap / g.s, kt = g.s - 1 - tap % g.s;
  const int src_tap = kr * g.s + kt;
  T (*tile)[33] = reinterpret_cast<T (*)[33]>(scratch);
  const T* fw = static_cast<const T*>(g.flip_w);
  T* fwt = static_cast<T*>(g.flip_wt);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int i = ty; i < 32; i += 8) {
    const int co = co0f + i, ci = ci0f + tx;
    tile[i][tx] = (co < g.cout && ci < g.cin) ? fw[((size_t)co * g.r * g.s + src_tap) * g.cin + ci] : T(0);
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int ci = ci0f + i, co = co0f + tx;
    if (ci < g.cin && co < g.cout) fwt[((size_t)ci * g.r * g.s + tap) * g.cout + co] = tile[tx][i];
  }
}

}  // namespace acc
