// What the bf16 matrix-core kernels share: the matrix instruction, loads from memory straight into LDS, and the order of their rows there.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace acc {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ __forceinline__ v16f mfma_bf16(const v4u& a, const v4u& b, v16f c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
#else
  return c;  // the host pass never runs this
#endif
}

template <int N> __device__ __forceinline__ void wait_loads() {      // at most N loads of the wave still on their way
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(N < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);  // and every LDS access done
#endif
}

// A buffer descriptor: `bytes` from p on, what lies outside reads as zero.
typedef unsigned srsrc __attribute__((ext_vector_type(4)));
__device__ __forceinline__ srsrc descriptor(const void* p, size_t bytes) {
  const uint64_t at = reinterpret_cast<uint64_t>(p);
  return srsrc{(uint32_t)at, (uint32_t)(at >> 32) & 0xffffu, (uint32_t)bytes, 0x00020000u};
}

// 16 bytes per lane from memory (soff the same for all) to LDS, lane l's to at + 16 * l.  Written out, because before a transposing LDS
// read the compiler waits for every such load it knows of, those of later chunks too; the kernels count them (wait_loads).  No register
// receives anything.  One wait state between writing m0 and an LDS load that reads it.  m0 cannot be declared: it is the compiler's own, which
// sets it for its builtins' loads into LDS and may set it once for several of them.  So a kernel has its loads into LDS either all from here or
// all from the builtin, and nothing else that needs m0.
__device__ __forceinline__ void load_lds16(srsrc rs, uint32_t voff, uint32_t soff, uint32_t at) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" : : "s"(at), "v"(voff), "s"(rs), "s"(soff) : "memory");
#endif
}
__device__ __forceinline__ void load_lds16(srsrc rs, uint32_t voff, uint32_t at) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(at), "v"(voff), "s"(rs) : "memory");
#endif
}

// Rows of PITCH bytes that the LDS read transposes: the 64-byte pieces of a row are XORed with this, so that the four rows that sixteen lanes
// read 32 bytes of each lie on different banks.  The same for rows a multiple of four apart.
template <int PITCH> __device__ __forceinline__ int row_xor(int row) { return PITCH == 64 ? 0 : PITCH == 128 ? (row >> 1) & 1 : row & 3; }

}  // namespace acc
